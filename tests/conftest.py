import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_sessionstart(session):
    """The tests load the library that is built in-tree; it is compiled here only when something is missing."""
    from paper_2605_18739_amd import build as hip_build
    if not (os.path.exists(hip_build.LIB) and os.path.exists(hip_build.HOST)):
        hip_build.build(verbose=False)


@pytest.fixture(scope="session")
def oracle():
    from oracle import nvfp4_oracle
    nvfp4_oracle.build()
    return nvfp4_oracle


@pytest.fixture(autouse=True, scope="session")
def _poison_fresh_nvfp4_outputs():
    """Every NVFP4 output tensor the binding allocates starts as 0xEE bytes during the tests (a
    scale byte no quantizer emits, and codes that differ from almost any result), so a byte that a
    kernel failed to write cannot pass for a correct one left over in recycled device memory."""
    from paper_2605_18739_amd import binding
    plain_init = binding.NVFP4Tensor.__init__

    def poisoned_init(self, rows, K, device="cuda", codes=None, scales=None, global_scale=None):
        plain_init(self, rows, K, device, codes, scales, global_scale)
        if codes is None:
            self.codes.fill_(0xEE)
        if scales is None:
            self.scales.fill_(0xEE)
        if global_scale is None:
            self.global_scale.fill_(float("nan"))

    binding.NVFP4Tensor.__init__ = poisoned_init
    yield
    binding.NVFP4Tensor.__init__ = plain_init

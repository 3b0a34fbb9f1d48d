import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU")
    config.addinivalue_line("markers", "slow: longer CPU test")


@pytest.fixture(scope="session")
def orc():
    import oracle
    oracle.lib()
    return oracle


@pytest.fixture(autouse=True)
def launches_end_with_the_test(request):
    """A GPU test may set or tune launch configurations; afterwards each is what
    it was before, so that every test starts from the shipped defaults whatever
    ran before it (a configuration holds for a power-of-two range of sizes)."""
    if request.node.get_closest_marker("gpu") is None:
        yield
        return
    import torch
    if not torch.cuda.is_available():
        yield
        return
    from paper_2605_04178_amd import wavemodel as wm
    ops = (wm.OP_PREDICT, wm.OP_VJP, wm.OP_LOSS_GRAD, wm.OP_SELECT_TILE, wm.OP_CALIBRATE_BATCHED, wm.OP_PREDICT_APPS,
           wm.OP_APPS_LOSS_GRAD)
    before = {(op, 1 << b): wm.get_launch(op, 1 << b) for op in ops for b in range(31)}
    yield
    for (op, n), c in before.items():
        if wm.get_launch(op, n) != c:
            wm.set_launch(op, n, **c)

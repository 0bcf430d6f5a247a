"""The hub push on the shapes of test_hub_push_exact, with the threshold of hub
slots below which it is off by itself taken away: six hub rows, every row a hub
row, and a row of 2^16 slots, for which the push is refused (its counters have
16 bits); then the no-allocation path, which pulls, on a plan with the push."""
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

from test_gpu_fw import test_hub_push_exact as _exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,iters", [("hubs", 1), ("hubs", 60), ("all_hubs", 1), ("all_hubs", 40),
                                         ("star", 1), ("star", 40)])
def test_pushed(shape, iters, monkeypatch):
    monkeypatch.setenv("LDS_PUSH_SLOTS", "0")
    _exact(shape, iters)

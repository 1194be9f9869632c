"""The tracking chain at the most frames of a launch, one fewer and one more
(its arrays full, and a second launch that goes on from their end), against the
oracle's tracker."""
import pytest

from test_gpu_chain import BASE, _check, _wander

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [255, 256, 257])
def test_largest_launch(n):
    _check(_wander(n, 192, 64, seed=n), 256, dict(BASE, track_radius=24, click_debounce=2))

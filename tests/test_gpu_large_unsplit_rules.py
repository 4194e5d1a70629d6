"""Fixed steps with stop rules at sizes that run one body a lane with no partners
shared (the layout of fixed steps without them shares), against the oracle."""
import pytest

from tests import test_gpu_large_rule_layouts as layouts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count", [(20, 3999), (80, 1000), (128, 1001), (400, 8), (512, 3)])
def test_unsplit_parity(fb, ora, n, count):
    layouts.test_rule_layout_parity(fb, ora, n, count, 0, 3)

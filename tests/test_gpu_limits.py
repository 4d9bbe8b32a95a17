"""The gradient of the largest training tiles, whose layers run on the marching kernel where
they have 60 and more output nodes a row."""
import pytest

from tests import test_gpu_network as network
from tests.test_gpu_surrogate import lbfd  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


# first layers of 58, 59, 63 and 70 output nodes a row; 64 is the largest tile
@pytest.mark.parametrize("T,B", [(52, 1), (53, 1), (57, 1), (64, 1)])
def test_gradient_of_large_tiles(lbfd, T, B):  # noqa: F811
    network.test_gradient_sizes(lbfd, T, B)

"""Launches that encode one vector a unit -- a query without a group, one key -- in every width of code, a unit without a new key among them."""
import pytest

pytestmark = pytest.mark.gpu

from tests.test_gpu_stage_ranges import test_encode_few_vectors as encode_few


@pytest.mark.parametrize("r", [32, 64, 96, 128, 192, 256])
@pytest.mark.parametrize("G", [1, 4])
def test_encode_one_vector(r, G):
    encode_few(r, G, 1)

"""GPU parity of the NetFlow v5 decode about the number of blocks whose totals a
decode workgroup sums itself (2,048; beyond, a scan kernel does).  Whole
numbers: tolerance 0."""
import pytest

from tests import test_gpu_ingest_tiles as tiles
from tests.test_gpu_ingest import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2048 * 1024, 2048 * 1024 + 1])
def test_blocks_summed_by_the_decode(torch_cuda, n):  # noqa: F811
    tiles.test_more_blocks_than_a_workgroup_sums(torch_cuda, n)

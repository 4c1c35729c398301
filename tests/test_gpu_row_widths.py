"""Every call on rows at the edges of the row copies' and folds' slices (one
chunk per lane up to 64 chunks of 16 bytes, three from 129 to 192, else two),
with fewer and more slots than folding waves, packs of one and two rows per
wave, and rows of many slices, bit for bit against the oracle."""
import pytest
import torch

import test_gpu_random_shapes as shapes
from paper_2609_36959_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    B.lib()
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("nch", [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 384, 512,
                                 640, 896, 2049, 2176])
@pytest.mark.parametrize("K,N", [(1, 3), (2, 2), (3, 2), (7, 3), (8, 3), (16, 9)])
def test_row_width(nch, K, N):
    shapes.test_random_shape(N, 2, 18 if N != 2 else 20, 18, K, 37, 8 * nch, "ragged", nch + K)

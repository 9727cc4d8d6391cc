"""Device memory that a plan takes (GPU): the workspace of marching by halves
only where a sweep of the plan marches."""
import numpy as np
import pytest

from tests.helpers import FIELDS, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles,least,most", [(None, 0, 3), ("lanes=1", 0, 3 + 7),
                                              ("lanes=0", 7, 3 + 8)])
def test_workspace_of_marching_by_halves(tiles, least, most):
    # 256 x 126 pencils along x, 106 x 126 and 106 x 256 along y and z, 240 bytes each:
    # 7.7, 3.2 and 6.5 MB, of which a plan keeps the largest that it marches; 3 MB for
    # its tables and the granularity of an allocation
    import torch
    from paper_1307_2265_amd import ppm
    dims = (100, 250, 120)
    shape = tuple(n + 6 for n in dims[::-1])
    patch = to_device({f: np.ones(shape) for f in FIELDS}, ppm.PPM_FP64)
    ppm.Plan([patch], 1, ppm.PPM_FP64, ppm.params(), tile_config=tiles).close()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    plan = ppm.Plan([patch], 1, ppm.PPM_FP64, ppm.params(), tile_config=tiles)
    torch.cuda.synchronize()
    taken = (before - torch.cuda.mem_get_info()[0]) / 2 ** 20
    plan.close()
    assert least <= taken <= most, taken

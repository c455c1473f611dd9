"""Zero-skipping launches with few tiles: the wavefronts of a workgroup share a tile's input channels, also shares that
are no whole channel blocks.  Every test here needs an MI355X."""
import pytest
import torch

import stgen
from oracle.st_ref import Geom

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests.gpu_harness import check_all_passes_full

# channel counts around the shares of 8 and 16 wavefronts: two channels each, uneven ones, one block split over several
# shares, shares that end inside a block; 1x1 with fewer, as many and more blocks than shares; stride 2
GEOMS = [Geom(1, 16, 16, 8, 8, 3, 3, 1, 1, 1, 1), Geom(1, 32, 48, 5, 9, 3, 3, 1, 1, 1, 1), Geom(2, 48, 16, 7, 7, 3, 3, 1, 1, 1, 1),
         Geom(1, 80, 128, 9, 10, 3, 3, 1, 1, 1, 1), Geom(1, 112, 272, 6, 14, 3, 3, 1, 1, 1, 1), Geom(1, 48, 80, 9, 11, 3, 3, 2, 2, 1, 1),
         Geom(1, 16, 80, 7, 9, 1, 1), Geom(1, 112, 48, 6, 6, 1, 1), Geom(2, 208, 256, 5, 7, 1, 1)]


@pytest.mark.parametrize("g", GEOMS, ids=[f"{g.R}x{g.S}/{g.stride_w} {g.C}to{g.K}" for g in GEOMS])
@pytest.mark.parametrize("dead", [0.0, 0.6])
def test_channel_shares_of_small_launches(g, dead):
    x = stgen.relu_sparse(g.x_shape, 0.5, 404)
    w = stgen.he_normal(g.w_shape, 405)
    dy = stgen.bernoulli_masked(g.y_shape, 0.5, 406, 407)
    if dead:
        x, dy = stgen.dead_channels(x, dead, 408), stgen.dead_channels(dy, dead, 409)
    check_all_passes_full(g, x, w, dy, "shares", variants=(False,))

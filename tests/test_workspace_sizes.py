"""Host-only: what the workspace of an fp32 pass holds besides the two feature maps -- the filters of the blocks that take the tile form
(block_tile.hip) show in its size."""
import pytest

import paper_1901_05350_amd as tfx
from paper_1901_05350_amd import binding


def beside_the_maps(size, q, batch):
    half = (size + 1) // 2
    return tfx.tfx_mobilenet_v1_variant_workspace_bytes(binding.TfxVariant(size, q, 1000), batch) - 2 * 4 * batch * half * half * 16 * q


# 512 -> 512 is a megabyte
@pytest.mark.parametrize("size,q,batch,tiles", [(64, 4, 2, False), (64, 4, 16, False), (128, 4, 4, False), (64, 3, 8, False), (224, 3, 3, False),
                                                (160, 2, 4, False), (224, 4, 8, True), (224, 4, 64, True), (160, 4, 24, True), (224, 3, 16, True)])
def test_small_passes_take_no_tiles(size, q, batch, tiles):
    """The tile form is slower than two launches for few outputs."""
    assert (beside_the_maps(size, q, batch) > 2 << 20) == tiles

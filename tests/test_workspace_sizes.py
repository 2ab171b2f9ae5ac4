"""Host-only: what the workspace of an fp32 pass holds besides the two feature maps -- the filters of the blocks that take the tile form
(block_tile.hip) show in its size."""
import ctypes

import pytest
import torch

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


def test_a_larger_batch_never_needs_less():
    for q in (1, 2, 3, 4):
        for size in (32, 33, 64, 65, 96, 128, 161, 224, 256):
            sizes = [tfx.tfx_mobilenet_v1_variant_workspace_bytes(binding.TfxVariant(size, q, 10), b) for b in range(2, 1025)]
            assert sizes == sorted(sizes), (q, size)


@pytest.mark.skipif(torch.cuda.is_available(), reason="calls the entry point on addresses that no GPU has")
def test_the_static_array_is_no_limit_of_other_workspaces():
    """A pass that fits the static array only without its filters has them in a workspace of its own."""
    size, batch = 33, 88
    assert beside_the_maps(size, 4, batch) > 2 << 20
    assert tfx.tfx_mobilenet_v1_variant_workspace_bytes(binding.TfxVariant(size, 4, 10), batch) > tfx.tfx_mobilenet_v1_static_scratch_bytes()
    w = binding.TfxWeights()
    for name in ("conv0_w", "conv0_b", "fc_w", "fc_b"):
        setattr(w, name, 0x1000)
    for name in ("dw_w", "dw_b", "pw_w", "pw_b"):
        for i in range(13):
            getattr(w, name)[i] = 0x1000
    fake = ctypes.c_void_p(0x1000)
    static = tfx.lib().tfx_mobilenet_v1_variant_forward_static
    assert static(ctypes.byref(binding.TfxVariant(size, 4, 10)), fake, batch, ctypes.byref(w), fake, None, None) == -6  # (no GPU)
    assert static(ctypes.byref(binding.TfxVariant(size, 4, 10)), fake, 2 * batch, ctypes.byref(w), fake, None, None) == -5

"""Host-only: a binary16 workspace serves one image, whatever batch it was sized for."""
import ctypes

import paper_1901_05350_amd as tfx
from paper_1901_05350_amd import binding


def test_one_image_fits_every_workspace():
    size_of = tfx.lib().tfx_mobilenet_v1_workspace_bytes_f16
    for q in (1, 2, 3, 4):
        for size in (32, 33, 64, 97, 128, 161, 224, 256):
            for classes in (1, 10, 1000, 1024):
                v = binding.TfxVariant(size, q, classes)
                sizes = [size_of(ctypes.byref(v), n) for n in (1, 2, 3, 4, 8, 16, 64)]
                assert sizes[0] > 0 and min(sizes) == sizes[0], (q, size, classes)

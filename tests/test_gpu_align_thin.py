"""The alignment's walk where a plane of the target takes at most half a block, so that several
walks share one: planes that fill it exactly or leave threads over, fewer planes than walks, a last
walk cut short.  Bounds as in test_gpu_align_walk."""

import pytest

import test_gpu_align_walk as walk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1000, 8, 8), (64, 16, 8), (50, 11, 11), (3, 2, 2), (201, 1, 7),
                                   (97, 1, 1)])
@pytest.mark.parametrize("whole", [True, False])
def test_thin_planes(shape, whole):
    walk.test_align_walk(shape, whole)

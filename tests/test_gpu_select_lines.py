"""Selection on both sides of the sizes where it takes several workgroups (4,096) and four
Gaussians per thread again (32,768)."""
import pytest

from tests import test_gpu_scene_kernels as K

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("n,pad", [(4097, 3), (4100, 0), (32_767, 1), (32_768, 0), (32_769, 3), (32_772, 0)])
def test_select_at_its_lines(R, orc, n, pad):
    K.test_select_sizes_and_alignment(R, orc, n, pad, 0, "f16")

"""What the library settles on the host before it launches anything: workspace sizes (no GPU needed)."""
import pytest

from paper_1804_04512_amd import binding as B
from paper_1804_04512_amd.workloads import ConvSpec


@pytest.mark.parametrize("shape", [(256, 1, 64, 64, 8, 3, 3, 1), (64, 1, 28, 28, 40, 9, 9, 0), (16, 3, 32, 32, 16, 5, 5, 2),
                                   (128, 16, 24, 24, 32, 3, 3, 1), (2, 1, 9, 9, 4, 4, 4, 0)])
def test_crbm_workspace_ignores_pooling_and_activation(shape):
    """The CRBM step ignores the descriptor's activation and pooling mode: it needs the same bytes whatever they
    are (a size taken from the pooled layer's plan was up to 1 MB short of what the step writes)."""
    sizes = {B.dll_crbm_workspace_bytes(ConvSpec(*shape, act, pool)) for act in ("identity", "relu") for pool in (1, 2)}
    assert len(sizes) == 1 and sizes.pop() > 0

"""bf16 attention backward: forms of the launch that the other attention tests do not reach, on their inputs and bounds."""
import pytest

import test_gpu_attention_modes as M

pytestmark = pytest.mark.gpu


# 56 pairs of 2 blocks: two launches in 64-row workgroups (no mask); 40: one launch of five pairs an XCD; 130: one launch in groups
# of 16 pairs and one, of which two XCDs have a pair
@pytest.mark.parametrize("b,h,causal", [(8, 7, False), (8, 5, True), (10, 13, True)])
@pytest.mark.parametrize("d", [64, 96, 128, 192])
@pytest.mark.parametrize("p_drop", [0.0, 0.1])
def test_backward_forms(b, h, causal, d, p_drop):
    M.test_attention_modes(b, h, d, causal, p_drop)

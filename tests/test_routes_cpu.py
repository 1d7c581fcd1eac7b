"""Which kernel the library takes, at sizes where both candidates were measured (times in the sources, beside the rules)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import routes  # noqa: E402


# direct path, channel counts that 256-wide blocks divide, one or more full rounds of 256x256 blocks: their kernel, up to the number of
# stages (of 64 channels, per tap) from which smaller blocks are level
@pytest.mark.parametrize("N,C,K,H,W,R,st,nhwc,wide", [
    (1, 128, 512, 256, 256, 1, 1, True, True), (1, 512, 1024, 256, 256, 1, 1, True, True), (1, 128, 1024, 128, 128, 3, 1, True, True), (1, 256, 512, 512, 512, 3, 2, True, True),
    (1, 256, 256, 512, 512, 3, 1, True, True), (1, 256, 256, 512, 512, 1, 1, True, True), (1, 1024, 1024, 128, 128, 3, 1, True, False),
    (1, 256, 240, 512, 512, 3, 1, True, False), (1, 256, 264, 512, 512, 1, 1, True, False), (1, 256, 256, 240, 240, 3, 1, True, False), (1, 512, 512, 180, 180, 3, 1, True, False),
    (1, 1024, 768, 180, 180, 3, 1, True, False), (1, 128, 768, 180, 180, 1, 1, True, True),
    (1, 64, 256, 256, 256, 3, 1, False, True), (1, 64, 1024, 180, 180, 3, 1, False, True), (1, 320, 1024, 256, 256, 1, 1, False, True), (1, 1024, 512, 256, 256, 1, 1, False, True),
    (1, 1024, 1024, 128, 128, 3, 1, False, False), (1, 64, 512, 180, 180, 3, 1, False, False), (1, 320, 320, 256, 256, 1, 1, False, False)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_direct_path_wide_blocks(N, C, K, H, W, R, st, nhwc, wide, dtype):
    assert (routes.igemm_tile(N, C, K, H, W, R, st, dtype, nhwc)[0] < 0) == wide

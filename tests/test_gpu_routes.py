"""GPU parity at the edges of the dispatch rules: the smallest and largest shapes of each kernel variant, ragged tiles,
workgroups that walk over several tiles and images.  Oracle, bar and protocol are those of test_gpu_parity.py."""
import pytest

import test_gpu_parity as base
from paper_2205_14756_amd import workloads as wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
# long contractions: a workgroup walks two tiles that belong to different images (70 ragged tiles, 64 workgroups a channel
# block), 24 and 32 chunks of weights; one whose last head-branches are missing in some waves (33)
@pytest.mark.parametrize("B,C,H,W,heads,scales", [(5, 512, 13, 33, 24, (5,)), (5, 512, 13, 33, 32, (5,)),
                                                  (2, 272, 9, 40, 11, (3, 5))])
def test_long_contraction_walks_tiles_of_several_images(dtype, B, C, H, W, heads, scales):
    print(f"routes: long contraction {dtype} {B}x{C}x{H}x{W} heads={heads}", flush=True)
    base.check_module(wk.random_module(41 + heads, dtype, B, C, H, W, heads, 16, scales), dtype, heads, 16, scales, stages=False)

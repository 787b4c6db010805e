"""The sources whose digest marks a committed counter figure as current: the kernel's own file, and the
headers with its device code and its tile rule."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def test_a_digest_covers_the_kernel_its_headers_and_its_tile_rule():
    for key, src in (("resblock_bwd/bf16/16x16/42x42", "resbwd.hip"), ("resblock_fwd/bf16/32x32/21x21", "resblock.hip"),
                     ("conv_bwd/bf16/64x64/21x21/relu/add", "convbwd.hip")):
        assert {src, "common.h", "kernels.h", "walk.h", "walkplan.h"} <= set(bench.source_files(key)), key
    assert {"convpool.hip", "common.h"} <= set(bench.source_files("conv_pool/bf16/4x16/84x84/u8"))
    assert bench.source_digest("resblock_bwd/bf16/16x16/42x42") != bench.source_digest("conv_pool/bf16/4x16/84x84/u8")
    assert bench.source_digest("no_such_family/bf16") is None

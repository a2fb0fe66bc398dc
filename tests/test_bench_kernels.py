"""The benchmark's own lists against the library (no GPU needed)."""
import glob
import os
import re

import bench
from paper_2505_20334_amd import binding


def test_every_scoring_kernel_is_counted_and_named(repo_root):
    csrc = os.path.join(repo_root, "paper_2505_20334_amd", "csrc")
    names = set()
    for path in glob.glob(os.path.join(csrc, "laq_score_*.hip")) + [os.path.join(csrc, f) for f in ("laq_head.hip", "laq_pool.hip")]:
        names |= set(re.findall(r"__global__[^;{]*?void\s+(\w+_kernel)\s*\(", open(path).read()))
    assert {"wave_stats_kernel", "tile_score_kernel", "fused_kernel", "head_kernel", "pool_quads_kernel"} <= names
    missed = [n for n in names if not any(k in n for k in bench.SCORE_STAGE_KERNELS)]
    assert not missed, missed
    assert set(bench.SCORE_KERNEL_TEXT) == set(binding.SCORE_KERNELS)
    for text in bench.SCORE_KERNEL_TEXT.values():
        named = re.findall(r"\w+_kernel\b", text)
        assert named and set(named) <= names, text

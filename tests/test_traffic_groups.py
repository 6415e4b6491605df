"""The groups of kernels that HBM bytes are counted for (traffic.py) against the kernels in the sources."""
import glob
import os
import re

from paper_2105_00619_amd import traffic as T

CSRC = os.path.join(os.path.dirname(os.path.abspath(T.__file__)), "csrc")


def test_every_convolution_and_batchnorm_kernel_is_in_one_group():
    text = "".join(open(f).read() for f in sorted(glob.glob(os.path.join(CSRC, "*.hip"))))
    kernels = set(re.findall(r"__global__ void[^;{]*?\b(\w+_kernel)\(", text))
    assert len(kernels) > 50
    counted = {k for k in kernels if k.startswith(("conv", "again_", "bn_apply", "bn_bwd", "wgrad_", "splitk_", "partial_"))}
    assert {"conv3x3_wide_kernel", "again_stats_kernel", "bn_bwd_apply_kernel"} <= counted
    for k in sorted(counted):
        groups = [g for g, fragments in T.GROUP_KERNELS.items() if any(f in "void oseq::(anonymous namespace)::%s<" % k for f in fragments)]
        assert len(groups) == 1, (k, groups)

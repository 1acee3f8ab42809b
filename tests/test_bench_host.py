"""CPU tests of what bench.py reads from committed files."""
import os

import pytest

import bench


@pytest.mark.parametrize("kind,kernel", sorted(bench.KIND_KERNEL.items()))
def test_kernel_names_are_in_the_committed_summary(kind, kernel):
    """A figure of the kernel statistics is looked up by the kernel's name there."""
    path = os.path.join(bench.ROOT, "profiles", "kernel_stats_ppd512.txt")
    with open(path) as f:
        assert sum(line.startswith(kernel + " ") for line in f) == 1, kernel

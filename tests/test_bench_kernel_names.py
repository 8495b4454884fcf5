"""Which dispatches of a profile belong to a kernel that the bench line names."""
from __future__ import annotations

import pytest

import bench


@pytest.mark.parametrize("kernel,name,match", [
    ("batch_step<0>", "void bcx::batch_step<0>(bcx::BatchArgs)", True),
    ("batch_step<0>", "void bcx::batch_step<1>(bcx::BatchArgs)", False),
    ("block_run<0>", "void bcx::block_run<0, 16>(bcx::BlockArgs)", True),
    ("block_run<0>", "void bcx::block_run<0>(bcx::BlockArgs)", True),
    ("block_run<0>", "void bcx::block_run<1, 16>(bcx::BlockArgs)", False),
    ("block_run<1>", "void bcx::block_run<16, 1>(bcx::BlockArgs)", False),
    ("wide_step<0>", "void bcx::batch_step<0>(bcx::BatchArgs)", False),
])
def test_kernel_names(kernel, name, match):
    assert bench._kernel_match(name, kernel) == match

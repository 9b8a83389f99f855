"""Transfer rows of more than 512 levels, which take a workgroup of the long
rows (those of more than 32 nodes) more than one pass."""

import pytest

import test_gpu_transfer_rows as rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nz", [(3, 175), (4, 130)])
def test_rows_of_many_levels_match_oracle(N, nz):
    rows.test_transfer_rows_match_oracle(N, nz)

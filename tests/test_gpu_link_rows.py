"""Linking table: it is emptied in the middle of a row (stretches of nearly
all distinct blocks), rows span several short stretches, stretches outlast a
wavefront's elements, and lengths on both sides of where those double."""
import pytest

from tests.test_gpu_load_partition import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,u", [(511, 511), (60_000, 60_000), (131_073, 100_000), (300_000, 30), (300_000, 1500),
                                 (4_194_303, 900_000), (4_194_304, 2_000_000)])
def test_rows(oracle_mod, n, u):
    check(oracle_mod, n, u, groups=2, skew=0.05, seed=3)

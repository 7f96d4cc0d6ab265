"""Extraction and selection at the edges between the forms for long rows and for many vectors: exact against the oracle."""
import pytest

from test_gpu_parity import test_extract_kept_columns_bit_exact as check_extraction, torch_mod, zr  # noqa: F401  (fixtures)
from test_gpu_select_lengths import test_many_vectors as check_many, torch_zr  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n", [(33, 5000), (18, 7000), (9, 12288), (5, 12296)])
def test_extraction_of_long_rows(zr, torch_mod, oracle, rows, n):  # noqa: F811
    check_extraction(zr, torch_mod, oracle, rows, n)


@pytest.mark.parametrize("kind", ["close", "wide", "ties"])
@pytest.mark.parametrize("n", [2048, 2049, 6144, 6145, 8192, 8193])
def test_many_vectors_of_one_length(torch_zr, kind, n):  # noqa: F811
    check_many(torch_zr, kind, 512, n)

"""Lists long enough for 32 slices in the attention that reads the pool (more than 16 slices of rows where there are
256 lists or more, four times that with fewer), at the edges of slices and of the limit, with the bounds of
test_gpu_row_slices."""
import pytest

from test_gpu_row_slices import check, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,slice_rows", [("f16", 128, 128), ("f32", 128, 128), ("f16", 64, 256)])
def test_few_long_lists(ctx, dtype, d, slice_rows):  # noqa: F811
    N = 64 * slice_rows + 100
    edges = [0, 1, 15 * slice_rows, 16 * slice_rows - 1, 16 * slice_rows, 16 * slice_rows + 1, 17 * slice_rows,
             32 * slice_rows - 1, 32 * slice_rows, 32 * slice_rows + 1, 33 * slice_rows, N]
    check(ctx, dtype, d, N, True, edges, N)


@pytest.mark.parametrize("dtype,d,slice_rows,new_row", [("f16", 128, 128, True), ("f16", 32, 512, False)])
def test_many_long_lists(ctx, dtype, d, slice_rows, new_row):  # noqa: F811
    N = 16 * slice_rows + 52
    edges = [3, 16 * slice_rows - 1, 16 * slice_rows, 16 * slice_rows + 1, N] + [40] * 251
    check(ctx, dtype, d, N, new_row, edges, N)

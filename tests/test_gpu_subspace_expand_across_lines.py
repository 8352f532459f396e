"""The reconstruction with rows in registers where the output's rows are no whole cache lines (expand_kernel): every number of k
steps, last tiles that share one to 31 columns with the tile before, a single tile that is moved by one column, row blocks that
end early, workgroups that share a row block and workgroups that go from one to the next.  Oracle and bars are those of
test_gpu_subspace.py."""
import pytest

from paper_2601_02360_amd import binding as B
from test_gpu_subspace import Misplaced, check_stage_boundary

pytestmark = pytest.mark.gpu
FP32, X3 = B.SPLC_MATMUL_FP32, B.SPLC_MATMUL_BF16X3

# on both sides of the lines of expand_applies_across_lines: `taken`
SHAPES = [
    (X3, 1, 33, 33, True, False, True), (X3, 127, 65, 64, True, True, True), (X3, 129, 255, 65, False, False, True),
    (X3, 300, 129, 97, True, False, True), (X3, 513, 257, 129, False, True, True), (X3, 641, 290, 161, True, True, True),
    (X3, 130, 513, 193, True, True, True), (X3, 1, 323, 222, False, False, True), (X3, 2048, 1931, 224, True, True, True),
    (X3, 38300, 131, 66, True, True, True), (X3, 40000, 417, 40, True, True, False), (X3, 9000, 333, 70, False, False, False),
    (X3, 15500, 703, 155, False, False, True), (X3, 20000, 100, 99, True, False, True),
    (FP32, 1, 83, 81, True, False, True), (FP32, 129, 129, 100, True, True, True), (FP32, 3300, 1307, 161, False, True, True),
    (FP32, 200, 250, 193, True, True, True), (FP32, 640, 385, 255, True, False, False), (FP32, 39400, 449, 256, True, True, True),
    (FP32, 30000, 420, 129, True, False, True), (FP32, 30000, 420, 129, True, True, False), (FP32, 640, 321, 130, True, True, False)]


@pytest.mark.parametrize("mode,rows,d,k,use_perp,use_pos,taken", SHAPES)
def test_reconstruction(mode, rows, d, k, use_perp, use_pos, taken):
    assert (B.subspace_kernel_choice(B.SPLC_OP_RECONSTRUCT, rows, d, k, use_perp + use_pos, mode) == (128, 32)) == taken
    check_stage_boundary(rows, min(rows, 1000), d, k, 50, use_perp, use_pos, seed=rows + d + k, mode=mode)


@pytest.mark.parametrize("mode,rows,d,k", [(X3, 513, 257, 191), (X3, 2050, 1283, 34), (FP32, 3390, 1299, 82), (FP32, 129, 251, 250)])
def test_arrays_aligned_to_four_bytes_and_ids_outside_the_table(mode, rows, d, k):
    """Guard values around every array; token ids beyond both ends."""
    assert B.subspace_kernel_choice(B.SPLC_OP_RECONSTRUCT, rows, d, k, 2, mode) == (128, 32)
    place = Misplaced()
    check_stage_boundary(rows, 300, d, k, 77, True, True, seed=rows + d + k, mode=mode, place=place, outside_ids=True)
    place.check()

"""The first product of the subspace calls where a workgroup takes 64 rows with all columns (contract_kernel, split
products): both column counts of a wave, columns that end inside a lane's, reductions that end inside a step of 16, a round
of 64 and a pair of rounds, row blocks that end early, one and two rounds of workgroups, every set of tables.  Oracle and
bars are those of test_gpu_subspace.py."""
import pytest

from paper_2601_02360_amd import binding as B
from test_gpu_subspace import check_reproject, check_stage_boundary

pytestmark = pytest.mark.gpu

PROJECT = [
    (8300, 512, 128, True, True), (8257, 513, 65, True, True), (4300, 527, 66, False, False), (8300, 528, 127, True, False),
    (8300, 575, 97, False, True), (17000, 576, 126, False, False), (5500, 640, 192, True, True), (5441, 704, 129, False, False),
    (6000, 700, 130, True, False), (6000, 1001, 191, False, True), (5600, 1039, 161, True, True), (22400, 520, 133, True, True),
    (16384, 1536, 192, True, True), (5999, 2050, 170, False, False)]


@pytest.mark.parametrize("rows,d,k,use_perp,use_pos", PROJECT)
def test_projection(rows, d, k, use_perp, use_pos):
    check_stage_boundary(rows, 300, d, k, 77, use_perp, use_pos, seed=rows + d + k, mode=B.SPLC_MATMUL_BF16X3)


@pytest.mark.parametrize("vocab,d,k", [(4300, 514, 67), (6001, 770, 190), (32001, 2050, 170)])
def test_reprojection(vocab, d, k):
    rows = list(range(200)) + list(range(vocab - 300, vocab))
    check_reproject(vocab, d, k, seed=vocab + d + k, mode=B.SPLC_MATMUL_BF16X3, rows=rows)

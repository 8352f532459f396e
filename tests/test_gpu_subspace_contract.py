"""The first product of the subspace calls where a workgroup takes 64 rows with all columns (contract_kernel and
contract_fp32_kernel): both column counts of a wave, columns that end inside a lane's, reductions that end inside a step of 16, a round
of 64 and a pair of rounds, row blocks that end early, one and two rounds of workgroups, every set of tables.  Oracle and
bars are those of test_gpu_subspace.py."""
import pytest
import torch

from paper_2601_02360_amd import binding as B
from test_gpu_subspace import Misplaced, check_reproject, check_stage_boundary

pytestmark = pytest.mark.gpu
FP32, X3 = B.SPLC_MATMUL_FP32, B.SPLC_MATMUL_BF16X3


def all_columns(op, rows, d, k, tables, mode):
    return B.subspace_kernel_choice(op, rows, d, k, tables, mode) == (64, 0)


PROJECT = [
    (8300, 512, 128, True, True), (8257, 513, 65, True, True), (4300, 527, 66, False, False), (8300, 528, 127, True, False),
    (8300, 575, 97, False, True), (17000, 576, 126, False, False), (5500, 640, 192, True, True), (5441, 704, 129, False, False),
    (8300, 700, 130, True, False), (6000, 1001, 191, False, True), (5600, 1039, 161, True, True), (22400, 520, 133, True, True),
    (16384, 1536, 192, True, True), (5999, 2050, 170, False, False)]
# fp32 products: reductions that end inside four k, a share of 16, a round of 64 and a pair of rounds
FP32_PROJECT = [
    (11008, 1024, 129, True, True), (11073, 1537, 160, False, False), (11000, 1055, 130, True, False), (11008, 1568, 161, False, False),
    (11007, 1087, 191, False, True), (22600, 1088, 192, True, True), (9793, 1548, 193, True, False), (9800, 1599, 194, False, True),
    (16384, 1600, 222, True, True), (26300, 1298, 223, True, False), (16383, 2050, 255, True, True), (16384, 2048, 256, True, True)]


@pytest.mark.parametrize("mode,rows,d,k,use_perp,use_pos", [(X3,) + c for c in PROJECT] + [(FP32,) + c for c in FP32_PROJECT])
def test_projection(mode, rows, d, k, use_perp, use_pos):
    assert all_columns(B.SPLC_OP_PROJECT, rows, d, k, use_perp + use_pos, mode)
    check_stage_boundary(rows, 300, d, k, 77, use_perp, use_pos, seed=rows + d + k, mode=mode)


@pytest.mark.parametrize("mode,vocab,d,k", [(X3, 4300, 514, 67), (X3, 6001, 770, 190), (X3, 32001, 2050, 170), (FP32, 11000, 1537, 163),
                                            (FP32, 32001, 1538, 192)])
def test_reprojection(mode, vocab, d, k):
    assert all_columns(B.SPLC_OP_REPROJECT_PASS1, vocab, d, k, 0, mode)
    rows = list(range(200)) + list(range(vocab - 300, vocab))
    check_reproject(vocab, d, k, seed=vocab + d + k, mode=mode, rows=rows)


@pytest.mark.parametrize("mode,rows,d,k", [(X3, 8257, 513, 65), (X3, 8257, 699, 131), (FP32, 11007, 1087, 191), (FP32, 16383, 1549, 254)])
def test_arrays_aligned_to_four_bytes_and_ids_outside_the_table(mode, rows, d, k):
    assert all_columns(B.SPLC_OP_PROJECT, rows, d, k, 2, mode)
    place = Misplaced()
    check_stage_boundary(rows, 300, d, k, 77, True, True, seed=rows + d + k, mode=mode, place=place, outside_ids=True)
    place.check()


@pytest.mark.parametrize("d,k", [(1344, 170), (1537, 160), (1539, 192)])
def test_infinities_and_nan_stay_in_their_row_and_column(d, k):
    """fp32 products: a NaN in x makes its row NaN; an infinite last entry of a column of U its column, nothing else."""
    rows = 11008
    assert all_columns(B.SPLC_OP_PROJECT, rows, d, k, 0, FP32)
    g = torch.Generator(device="cuda").manual_seed(d)
    x = torch.rand(rows, d, generator=g, device="cuda") + 0.5
    u = torch.randn(d, k, generator=g, device="cuda")
    x[5, d - 1] = float("nan")
    x[130, 0] = float("inf")
    u[d - 1, k - 1] = float("inf")
    u[7, 64] = float("nan")
    out = torch.empty(rows, k, device="cuda")
    B.sparseloco_subspace_project(x, u, out, matmul=FP32)
    want = torch.zeros(rows, k, dtype=torch.bool, device="cuda")
    want[5], want[130], want[:, k - 1], want[:, 64] = True, True, True, True
    assert torch.equal(~torch.isfinite(out), want)
    assert torch.isnan(out[5]).all() and torch.isinf(out[131:, k - 1]).all() and torch.isnan(out[:, 64]).all()

"""The second product of the subspace calls where it keeps its rows in registers and walks along the columns
(expand_kernel): every number of k steps, reductions that end inside a group of four and inside a step, row blocks that
end early, workgroups that share a row block and workgroups that go from one to the next.  Oracle and bars are those of
test_gpu_subspace.py."""
import pytest
import torch

from paper_2601_02360_amd import binding as B
from test_gpu_subspace import Misplaced, check_reproject, check_stage_boundary

pytestmark = pytest.mark.gpu
FP32, X3 = B.SPLC_MATMUL_FP32, B.SPLC_MATMUL_BF16X3


def rows_in_registers(op, rows, d, k, tables, mode):
    return B.subspace_kernel_choice(op, rows, d, k, tables, mode) == (128, 32)


# split products: from one row on where the number of 64-column blocks is even, 1200 tiles of 128 x 32 where it is odd; k 33 ...
# 224 are two to seven steps of 32
X3_RECONSTRUCT = [
    (1, 256, 33, True, True), (127, 128, 64, True, False), (128, 256, 65, False, False), (129, 128, 96, False, True),
    (300, 128, 97, True, True), (1000, 256, 128, False, False), (257, 256, 129, True, True), (640, 256, 161, False, True),
    (130, 512, 191, True, False), (513, 256, 192, True, True), (129, 256, 193, False, False), (1, 256, 222, True, True),
    (2048, 1920, 224, True, True), (38300, 128, 66, True, True), (20000, 384, 99, False, False), (15400, 320, 131, True, False),
    (15500, 352, 155, False, False)]
# fp32 products: from 3072 tiles on (4096 without tables, 8192 for k above 224), three to eight steps
FP32_RECONSTRUCT = [
    (39300, 320, 81, True, True), (39400, 320, 96, True, False), (23900, 704, 100, True, False), (24500, 512, 127, False, True),
    (47700, 352, 128, False, False), (18900, 704, 161, True, True), (39400, 320, 192, True, True), (39350, 320, 223, True, True),
    (39400, 320, 256, True, True), (95400, 352, 253, False, False)]


@pytest.mark.parametrize("mode,rows,d,k,use_perp,use_pos", [(X3,) + c for c in X3_RECONSTRUCT] + [(FP32,) + c for c in FP32_RECONSTRUCT])
def test_reconstruction(mode, rows, d, k, use_perp, use_pos):
    assert rows_in_registers(B.SPLC_OP_RECONSTRUCT, rows, d, k, use_perp + use_pos, mode)
    check_stage_boundary(rows, min(rows, 1000), d, k, 50, use_perp, use_pos, seed=rows + d + k, mode=mode)


REPROJECT = [
    (X3, 1, 384, 33), (X3, 641, 64, 33), (X3, 128, 128, 64), (X3, 300, 128, 98), (X3, 1000, 320, 200), (X3, 129, 256, 224),
    (X3, 3000, 96, 40), (X3, 40000, 384, 40), (X3, 7000, 768, 96), (FP32, 196608, 64, 42), (FP32, 65537, 192, 67),
    (FP32, 49152, 256, 96), (FP32, 49100, 256, 129), (FP32, 49152, 256, 161), (FP32, 12300, 1024, 200), (FP32, 49152, 256, 255)]


def ends_and_middle(vocab):
    return sorted(set(range(min(vocab, 400))) | set(range(max(0, vocab - 400), vocab)) | set(range(vocab // 2, min(vocab, vocab // 2 + 300))))


@pytest.mark.parametrize("mode,vocab,d,k", REPROJECT)
def test_reprojection(mode, vocab, d, k):
    assert rows_in_registers(B.SPLC_OP_REPROJECT_PASS2, vocab, d, k, 0, mode)
    check_reproject(vocab, d, k, seed=vocab + d + k, mode=mode, rows=ends_and_middle(vocab))


@pytest.mark.parametrize("mode,rows,d,k", [(X3, 513, 256, 191), (X3, 2050, 1280, 34), (FP32, 39390, 320, 82), (FP32, 39390, 320, 255)])
def test_arrays_aligned_to_four_bytes_and_ids_outside_the_table(mode, rows, d, k):
    assert rows_in_registers(B.SPLC_OP_RECONSTRUCT, rows, d, k, 2, mode)
    place = Misplaced()
    check_stage_boundary(rows, 300, d, k, 77, True, True, seed=rows + d + k, mode=mode, place=place, outside_ids=True)
    place.check()


@pytest.mark.parametrize("mode,vocab,d,k", [(X3, 300, 128, 98), (X3, 2049, 640, 201), (FP32, 49100, 256, 129)])
def test_reprojection_of_arrays_aligned_to_four_bytes(mode, vocab, d, k):
    assert rows_in_registers(B.SPLC_OP_REPROJECT_PASS2, vocab, d, k, 0, mode)
    place = Misplaced()
    check_reproject(vocab, d, k, seed=vocab + d + k, mode=mode, rows=ends_and_middle(vocab), place=place)
    place.check()


@pytest.mark.parametrize("k", [81, 82, 83, 84])
def test_infinities_and_nan_stay_in_their_row_and_column(k):
    """fp32 products: a NaN row of coefficients makes that row NaN, an infinite entry of U its column, nothing else."""
    rows, d = 39424, 320
    assert rows_in_registers(B.SPLC_OP_RECONSTRUCT, rows, d, k, 1, FP32)
    g = torch.Generator(device="cuda").manual_seed(k)
    x = torch.randn(rows, k, generator=g, device="cuda")
    u = torch.randn(d, k, generator=g, device="cuda")
    x[5, 2] = float("nan")
    x[130, k - 1] = float("inf")
    u[7, 0] = float("inf")
    u[64, k - 1] = float("nan")
    pos = torch.zeros(16, d, device="cuda")
    out = torch.empty(rows, d, device="cuda")
    B.sparseloco_subspace_reconstruct(x, u, out, pos_embed=pos, matmul=FP32)
    bad = ~torch.isfinite(out)
    want = torch.zeros_like(bad)
    want[5], want[130], want[:, 7], want[:, 64] = True, True, True, True
    assert torch.equal(bad, want)
    assert torch.isnan(out[5]).all() and torch.isinf(out[130, 8:64]).all() and torch.isnan(out[:, 64]).all()

"""The second product of the subspace calls where it keeps its rows in registers and walks along the columns
(expand_kernel): every number of k steps, reductions that end inside a group of four and inside a step, row blocks that
end early, workgroups that share a row block and workgroups that go from one to the next.  Oracle and bars are those of
test_gpu_subspace.py."""
import pytest
import torch

from paper_2601_02360_amd import binding as B
from test_gpu_subspace import check_reproject, check_stage_boundary

pytestmark = pytest.mark.gpu
FP32, X3 = B.SPLC_MATMUL_FP32, B.SPLC_MATMUL_BF16X3

# split products take the kernel from one row on; k 33 ... 224 are two to seven steps of 32
X3_RECONSTRUCT = [
    (1, 256, 33, True, True), (127, 128, 64, True, False), (128, 256, 65, False, False), (129, 128, 96, False, True),
    (300, 128, 97, True, True), (1000, 256, 128, False, False), (257, 256, 129, True, True), (640, 256, 161, False, True),
    (130, 512, 191, True, False), (513, 256, 192, True, True), (129, 256, 193, False, False), (1, 256, 222, True, True),
    (2048, 1920, 224, True, True), (38300, 128, 66, True, True), (20000, 384, 99, False, False), (9800, 320, 131, True, False)]


@pytest.mark.parametrize("rows,d,k,use_perp,use_pos", X3_RECONSTRUCT)
def test_reconstruction_with_split_products(rows, d, k, use_perp, use_pos):
    check_stage_boundary(rows, min(rows, 100), d, k, 50, use_perp, use_pos, seed=rows + d + k, mode=X3)


# fp32 products from 3072 tiles of 128 x 32 on (4096 without tables, 8192 for k above 224)
FP32_RECONSTRUCT = [
    (131072, 96, 81, True, True), (65500, 192, 96, True, False), (49152, 256, 127, False, True), (65536, 256, 130, False, False),
    (49100, 256, 161, True, True), (49152, 256, 192, True, True), (49030, 256, 223, True, True), (49152, 256, 256, True, True),
    (131072, 256, 253, False, False)]


@pytest.mark.parametrize("rows,d,k,use_perp,use_pos", FP32_RECONSTRUCT)
def test_reconstruction_with_fp32_products(rows, d, k, use_perp, use_pos):
    check_stage_boundary(rows, 1000, d, k, 50, use_perp, use_pos, seed=rows + d + k, mode=FP32)


REPROJECT = [
    (X3, 1, 64, 33), (X3, 128, 64, 64), (X3, 300, 128, 98), (X3, 1000, 320, 200), (X3, 129, 256, 224), (X3, 40000, 96, 40),
    (X3, 7000, 768, 96), (FP32, 196608, 64, 34), (FP32, 65537, 192, 67), (FP32, 49152, 256, 96), (FP32, 49100, 256, 129),
    (FP32, 49152, 256, 161), (FP32, 12300, 1024, 200), (FP32, 49152, 256, 255)]


@pytest.mark.parametrize("mode,vocab,d,k", REPROJECT)
def test_reprojection(mode, vocab, d, k):
    ends = sorted(set(range(min(vocab, 400))) | set(range(max(0, vocab - 400), vocab)) | set(range(vocab // 2, min(vocab, vocab // 2 + 300))))
    check_reproject(vocab, d, k, seed=vocab + d + k, mode=mode, rows=ends)


@pytest.mark.parametrize("k", [81, 82, 83, 84])
def test_infinities_and_nan_stay_in_their_row_and_column(k):
    """fp32 products: a NaN row of coefficients makes that row NaN, an infinite entry of U its column, nothing else."""
    rows, d = 131072, 96
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

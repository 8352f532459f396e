"""Compression in strips of four tiles (compress_strip_kernel) on plans that take it: against the same compression tile by
tile, which compress_batch does on every plan and the oracle tests elsewhere cover, bit for bit.  Complete tiles left over
beside the strips, edge tiles below and to the right; among the strips some whose four tiles disagree about the path of the
selection.  Which plans take strips is splc::strips_pay's choice: check_strips_pay of launch_rules_main.cpp holds its lines
where this file needs them."""
import pytest
import torch

from paper_2601_02360_amd import binding as B

COLS = 1222                                       # 19 complete tiles: four strips, three tiles beside them, and 6 columns


def rows_of(strips):
    return 64 * (strips // 4) + 3


def delta_of(rows, seed, bf16):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(rows, COLS, generator=g, device="cuda") * 1e-3
    x *= 1 + 9 * (torch.rand(rows, COLS, generator=g, device="cuda") < 0.01)          # a heavy tail
    x[:64, 0:64] = -7.25                          # one strip: constant (a 4096-way tie), zero, few values, ordinary
    x[:64, 64:128] = 0.0
    x[:64, 128:192] = torch.randint(0, 3, (64, 64), generator=g, device="cuda") * 0.125
    x[64:128, 256 + 64:256 + 128] = 3.0           # one constant tile among ordinary ones
    x[128:192, 0:256] = 0.0                       # four that agree on the general path
    x[192:256, 0:256] = float("inf")
    return x.to(torch.bfloat16) if bf16 else x


@pytest.mark.gpu
@pytest.mark.parametrize("source,kappa,quant,select,strips", [
    ("params", 1, True, B.SPLC_SELECT_AUTO, 2700), ("params", 64, False, B.SPLC_SELECT_AUTO, 2700),
    ("params", 128, True, B.SPLC_SELECT_RADIX, 2700), ("params", 192, True, B.SPLC_SELECT_AUTO, 2700),
    ("f32", 32, True, B.SPLC_SELECT_AUTO, 6500), ("f32", 128, False, B.SPLC_SELECT_RADIX, 6500), ("f32", 192, False, B.SPLC_SELECT_AUTO, 6500),
    ("bf16", 64, True, B.SPLC_SELECT_RADIX, 6500), ("bf16", 32, False, B.SPLC_SELECT_AUTO, 6500),
    ("bf16", 128, True, B.SPLC_SELECT_AUTO, 6500), ("bf16", 160, False, B.SPLC_SELECT_AUTO, 6500)])
def test_strips_match_tile_by_tile(source, kappa, quant, select, strips):
    rows = rows_of(strips)
    table = B.chunk_table([(rows, COLS)], True)
    assert int((table["strip"] == 1).sum()) == strips
    delta = delta_of(rows, kappa, source == "bf16")
    n = delta.numel()
    e0 = torch.randn(n, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda") * 1e-4
    # theta_outer - theta_local = delta: what a call from parameters is given, and the one that goes tile by tile
    theta, local = delta.float().reshape(-1), torch.zeros(n, device="cuda")
    results = []
    for batched in (False, True):
        plan = B.Plan([(rows, COLS)], kappa, quant=quant, tiled=True)
        plan.set_select(select)
        e = e0.clone()
        pairs, aux = plan.message_buffers()
        pairs.fill_(0x5A5A), aux.fill_(float("nan"))
        if batched:
            B.sparseloco_compress_batch(plan, [theta], [[local]], [[e]], [pairs], 0.95, aux_out=[aux])
        elif source == "params":
            B.sparseloco_compress(plan, [e], pairs, aux, 0.95, theta_outer=[theta], theta_local=[local])
        else:
            B.sparseloco_compress(plan, [e], pairs, aux, 0.95, delta=[delta.reshape(-1)])
        torch.cuda.synchronize()
        results.append((pairs, aux.view(torch.int32), e.view(torch.int32)))
        plan.close()
    for got, want in zip(*results):
        assert torch.equal(got, want)

"""The aggregation's kernels: entries per lane (kappa up to 64, 128, 256 and more), batches of eight replicas with a last one
that is not full, a division by M that is a power of two or not (subnormal sums among them), and on plans of 8192 chunks and
more the orders in which theta and the messages are read.  The sum over replicas in order, formed with torch, is bit-exact."""
import pytest
import torch

from paper_2601_02360_amd import binding as B
from test_gpu_aggregate_runs import CHUNK, messages

pytestmark = pytest.mark.gpu


def check(numels, kappa, replicas, quant, tiny=False):
    total = sum(numels)
    mean = torch.zeros(total, device="cuda")
    pairs, aux = [], []
    for p, levels, position, value in messages(numels, kappa, replicas, seed=kappa + replicas):
        if tiny:                                 # every second position gets subnormal values
            small = position % 2 == 0
            value = torch.where(small, value * 2.0 ** -140, value)
        if not quant:
            sent = p != -1
            levels = torch.zeros(p.numel(), device="cuda")
            levels[sent] = value
            p = torch.where(sent, p & 0xFFF, p)
        pairs.append(p)
        aux.append(levels)
        mean[position] += value                  # a replica sends a position once
    mean = (mean.cpu() / replicas).cuda()
    theta = torch.randn(total, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    want = theta - 0.5 * mean
    plan = B.Plan(numels, kappa, quant=quant)
    received = plan.bind_messages(pairs, aux)
    got = torch.full_like(mean, float("nan"))
    B.sparseloco_aggregate(plan, received, plan.bind(list(got.split(numels))))
    assert torch.equal(got, mean)
    got.fill_(float("nan"))
    local = torch.full((2, total), float("nan"), device="cuda")
    B.sparseloco_aggregate_update(plan, received, plan.bind(list(theta.split(numels))), 0.5,
                                  delta_bar_out=plan.bind(list(got.split(numels))),
                                  reset=plan.bind([list(t.split(numels)) for t in local]))
    assert torch.equal(got, mean) and torch.equal(theta, want)
    assert torch.equal(local[0], want) and torch.equal(local[1], want)


@pytest.mark.parametrize("quant", [True, False])
@pytest.mark.parametrize("kappa", [1, 63, 64, 65, 128, 129, 256, 257])
@pytest.mark.parametrize("replicas", [1, 7, 8, 9, 32, 33])
def test_entries_and_batches(kappa, replicas, quant):
    check([CHUNK * 3 + 70, 5, CHUNK], kappa, replicas, quant, tiny=not quant)


@pytest.mark.parametrize("quant", [True, False])
@pytest.mark.parametrize("kappa", [65, 128, 129, 256, 257, 4096])
@pytest.mark.parametrize("replicas", [1, 4, 9, 33])
def test_chunks_of_fewer_elements_than_kappa(kappa, replicas, quant):
    """Each takes the way of its own messages: one, two or four entries per lane, or one replica after the other."""
    check([1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, CHUNK + 40, 4095], kappa, replicas, quant)


# With the update, theta late: 2 and 3; 9 of kappa 64; the unquantised ones (8 of kappa 64 and 128 in fewer groups a unit) / with the
# first messages: 9 of kappa 16; 2 of kappa 200.  (The lines: check_aggregate_pace of launch_rules_main.cpp.)
@pytest.mark.parametrize("kappa,replicas,quant", [(16, 3, True), (16, 9, True), (64, 9, True), (200, 2, True), (64, 8, False),
                                                  (128, 8, False), (32, 5, False), (16, 2, True)])
@pytest.mark.parametrize("chunks", [8191, 8192])
def test_large_plans(chunks, kappa, replicas, quant):
    check([CHUNK * (chunks - 2) + 100, 3], kappa, replicas, quant)


@pytest.mark.parametrize("cols", [2048, 2050])                  # rows of whole cache lines, or not
@pytest.mark.parametrize("kappa,replicas,quant", [(64, 3, False), (31, 9, True), (200, 17, True), (300, 7, False)])
def test_mean_of_tiles_with_stores_together(kappa, replicas, quant, cols):
    """Complete tiles, edge tiles and flat chunks of a large tiled plan, against the mean that the aggregation with outer update
    writes, whose divisions and stores take turns."""
    shapes = [(64 * (8320 // -(-cols // 64)) - 3, cols), (65, 2), (1, 4100)]
    table = B.chunk_table(shapes, True)
    chunks = len(table)
    assert chunks >= 8192
    plan = B.Plan(shapes, kappa, quant=quant, tiled=True)
    g = torch.Generator(device="cuda").manual_seed(kappa + replicas)
    slot = torch.arange(kappa, device="cuda")
    size = torch.empty(chunks, dtype=torch.int64)
    size[torch.from_numpy(table["id"].astype("int64"))] = torch.from_numpy(table["n_c"].astype("int64"))
    sent = slot < size.cuda()[:, None]
    pairs, aux = [], []
    for _ in range(replicas):
        step = torch.randint(0, CHUNK // 2, (chunks, 1), generator=g, device="cuda") * 2 + 1
        index = step * slot % CHUNK                             # distinct inside a message
        if quant:
            index = index + 4096 * torch.randint(0, 4, index.shape, generator=g, device="cuda")
        pairs.append(torch.where(sent, index, torch.full_like(index, 0xFFFF)).to(torch.int32).to(torch.int16).reshape(-1))
        aux.append(torch.randn(chunks * (2 if quant else kappa), generator=g, device="cuda"))
    received = plan.bind_messages(pairs, aux)
    numels = [r * c for r, c in shapes]
    got, want = (torch.full((sum(numels),), float("nan"), device="cuda") for _ in range(2))
    theta = torch.zeros_like(got)
    B.sparseloco_aggregate(plan, received, plan.bind(list(got.split(numels))))
    B.sparseloco_aggregate_update(plan, received, plan.bind(list(theta.split(numels))), 1.0,
                                  delta_bar_out=plan.bind(list(want.split(numels))))
    assert not got.isnan().any() and torch.equal(got.view(torch.int32), want.view(torch.int32))

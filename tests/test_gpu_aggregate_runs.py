"""The aggregation where every XCD takes runs of chunks: many replicas, quantised messages, at least 9000 chunks; whole
rounds of eight runs and places behind the last one, element-wise chunks among them.  The sum over replicas in order, formed
with torch, is bit-exact."""
import pytest
import torch

from paper_2601_02360_amd import binding as B

pytestmark = pytest.mark.gpu
CHUNK = 4096


def messages(numels, kappa, replicas, seed):
    """Pairs and levels of random messages, and per replica the positions (in all tensors laid end to end) and values sent."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    starts, sizes, first = [], [], 0
    for n in numels:
        for at in range(0, n, CHUNK):
            starts.append(first + at)
            sizes.append(min(CHUNK, n - at))
        first += n
    start, size = torch.tensor(starts, device="cuda")[:, None], torch.tensor(sizes, device="cuda")[:, None]
    slot = torch.arange(kappa, device="cuda")
    sent = slot < size
    for _ in range(replicas):
        at = torch.randint(0, CHUNK, size.shape, generator=g, device="cuda")
        step = torch.randint(0, CHUNK // 2, size.shape, generator=g, device="cuda") * 2 + 1
        index = torch.where(size == CHUNK, (at + step * slot) % CHUNK, slot).where(sent, torch.zeros_like(slot))
        flags = torch.randint(0, 4, index.shape, generator=g, device="cuda")
        levels = torch.rand(len(starts), 2, generator=g, device="cuda")
        value = torch.where(flags % 2 == 1, levels[:, 1:], levels[:, :1]) * torch.where(flags >= 2, -1.0, 1.0)
        pairs = torch.where(sent, index + 4096 * flags, torch.full_like(index, 0xFFFF))
        yield pairs.to(torch.int32).to(torch.int16).reshape(-1), levels.reshape(-1), (start + index)[sent], value[sent]


@pytest.mark.parametrize("numels,kappa,replicas", [
    ([CHUNK * 9000], 16, 32), ([CHUNK * 9080 + 230, 7, CHUNK * 2], 33, 24),
    ([CHUNK * 11999 + 1, CHUNK * 160], 64, 33)])
def test_every_chunk_once(numels, kappa, replicas):
    total = sum(numels)
    mean = torch.zeros(total, device="cuda")
    pairs, aux = [], []
    for p, levels, position, value in messages(numels, kappa, replicas, seed=kappa + replicas):
        pairs.append(p)
        aux.append(levels)
        mean[position] += value                  # a replica sends a position once
    mean = mean / torch.full_like(mean, replicas)
    theta = torch.randn(total, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    want = theta - 0.5 * mean
    plan = B.Plan(numels, kappa)
    got = torch.full_like(mean, float("nan"))
    received = plan.bind_messages(pairs, aux)
    B.sparseloco_aggregate(plan, received, plan.bind(list(got.split(numels))))
    assert torch.equal(got, mean)
    B.sparseloco_aggregate_update(plan, received, plan.bind(list(theta.split(numels))), 0.5)
    assert torch.equal(theta, want)

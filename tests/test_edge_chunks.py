"""Edge chunks, read four elements at a time by vectors that end at a lane's last present element: where those vectors
lie (on the CPU, the rule restated in numpy over the table of chunks), and the results against the oracle at widths,
heights and tails around the vectors' size."""
import numpy as np
import pytest
import torch

from paper_2601_02360_amd import binding as B

import parity

SHAPES = [(64, w) for w in (1, 2, 3, 4, 5, 7, 13, 29, 63)] + [(h, 66) for h in (1, 2, 15, 16, 17, 65)] + \
         [(130, 2), (65, 1), (1, 3), (2, 1), (70, 191), (129, 67), (66, 257)]
TAILS = [1, 2, 3, 4, 5, 63, 65, 66, 67, 1023, 1026, 4095, 4097, 4098, 4099, 8191]


@pytest.mark.parametrize("tiled", [False, True], ids=["flat", "tile"])
def test_vectors_of_edge_chunks_stay_inside_their_tensor(tiled):
    shapes = SHAPES if tiled else [(n,) for n in TAILS]
    tab = B.chunk_table(shapes, tiled)
    sizes = [int(np.prod(s)) for s in shapes]
    tid, slot = np.meshgrid(np.arange(256), np.arange(4))
    lr, lc = slot * 16 + tid // 16, tid % 16 * 4
    narrow_seen = 0
    for d in tab[tab["vec"] == 0]:
        h, w, last = int(d["h"]), int(d["w"]), int(d["last_w"])
        w0 = w if h > 1 else last
        width = np.where(lr + 1 < h, w, np.where(lr + 1 == h, last, 0))
        n = np.clip(width - lc, 0, 4)
        assert n.sum() == d["n_c"]
        end = np.where(n > 0, lr * int(d["stride"]) + lc + n, min(w0, 4))       # behind the last element read
        first = int(d["offset"]) + end - 4
        assert (int(d["offset"]) + end).max() <= sizes[d["tensor"]]
        if d["offset"] == 0 and w0 < 4:                     # narrow: read one by one, never below the first
            narrow_seen += 1
        else:
            assert first.min() >= 0
    assert narrow_seen


def case_of(shapes, tiled, R, seed, direct=None):
    rng = np.random.default_rng(seed)
    numels = [int(np.prod(s)) for s in shapes]
    th = [(rng.standard_normal(n) * 0.02).astype(np.float32) for n in numels]
    ef = [[(rng.standard_normal(n) * 1e-4).astype(np.float32) for n in numels] for _ in range(R)]
    deltas = [[(rng.standard_t(3, n) * 1e-3).astype(np.float32) for n in numels] for _ in range(R)]
    shapes = [tuple(s) for s in shapes] if tiled else None
    if direct == "bf16":
        return parity.HostCase(th, ef, delta=[[(x.view(np.uint32) >> 16).astype(np.uint16) for x in r] for r in deltas],
                               shapes=shapes)
    if direct:
        return parity.HostCase(th, ef, delta=deltas, shapes=shapes)
    return parity.HostCase(th, ef, theta_local=[[t - x for t, x in zip(th, r)] for r in deltas], shapes=shapes)


@pytest.mark.gpu
@pytest.mark.parametrize("how", [dict(), dict(direct="f32", quant=False, fused="with_mean"),
                                 dict(direct="bf16", fused="no_mean"), dict(batch=True, fused="with_mean")],
                         ids=["params", "f32", "bf16", "batch"])
@pytest.mark.parametrize("kappa", [1, 16, 64, 128, 256])
@pytest.mark.parametrize("tiled", [False, True], ids=["flat", "tile"])
def test_edge_chunks_match_the_oracle(tiled, kappa, how):
    how = dict(how)
    case = case_of(SHAPES if tiled else [(n,) for n in TAILS], tiled, 2, kappa, how.pop("direct", None))
    parity.check(case, kappa, outer_steps=2, what="edge chunks kappa=%d %s" % (kappa, how), **how)


@pytest.mark.gpu
@pytest.mark.parametrize("kappa,shape", [(128, (640, 5)), (128, (640, 13)), (128, (640, 28)), (64, (640, 9)), (256, (640, 40)), (128, (9, 640)), (64, (5, 640))])
def test_edge_tiles_of_few_lanes_take_the_candidate_filter(kappa, shape):
    """Tiles whose waves hold fewer elements than their equal share of kappa: distinct values, so the filter's bound has to
    keep the candidates few enough."""
    n = shape[0] * shape[1]
    g = torch.Generator(device="cuda").manual_seed(kappa + n)
    th, tl, ef = (torch.randn(n, generator=g, device="cuda") for _ in range(3))
    plan = B.Plan([shape], kappa, tiled=True)
    pairs, aux = plan.message_buffers()
    counter = torch.zeros(1, dtype=torch.int32, device="cuda")
    plan.set_radix_counter(counter)
    B.sparseloco_compress(plan, [ef], pairs, aux, 0.95, theta_outer=[th], theta_local=[tl])
    assert int(counter.item()) == 0


@pytest.mark.gpu
def test_what_lies_around_an_edge_chunk_is_left_alone():
    """Tensors back to back in one buffer, with guard values between them."""
    shapes = [s for s in SHAPES if s[0] > 1]
    sizes = [r * c for r, c in shapes]
    rng = np.random.default_rng(3)
    plan = B.Plan(shapes, 16, tiled=True)
    start = np.concatenate([[1], 1 + np.cumsum(np.array(sizes) + 1)])
    host = [(rng.standard_normal(int(start[-1])) * s).astype(np.float32) for s in (0.02, 0.02, 1e-4)]
    for h in host:
        h[start - 1] = 77.0
    bufs = [torch.from_numpy(h.copy()).cuda() for h in host]
    views = [[b[int(s):int(s) + n] for s, n in zip(start, sizes)] for b in bufs]
    pairs, aux = plan.message_buffers()
    B.sparseloco_compress(plan, views[2], pairs, aux, 0.95, theta_outer=views[0], theta_local=views[1])
    B.sparseloco_aggregate_update(plan, [pairs], views[0], 1.0, aux=[aux])
    for b in bufs:
        assert np.all(parity.to_np(b)[start - 1] == 77.0)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,direct,kappa", [(64 * 674, None, 32), (64 * 675 + 3, None, 128), (64 * 1624, "bf16", 64),
                                               (64 * 1625 + 3, "bf16", 64)])
def test_strips_and_tiles_on_both_sides_of_the_line(rows, direct, kappa):
    """Matrices of 1030 columns, four strips a tile row: the largest plan that is compressed tile by tile, and the
    smallest (with rows to spare) that takes strips."""
    case = case_of([(rows, 1030)], True, 1, kappa, direct)
    parity.check(case, kappa, fused="no_mean", what="%d rows kappa=%d" % (rows, kappa))

"""The native way of the binding's launching calls (csrc/calls.cpp): it makes the call or hands the arguments back, and
what it hands back is refused, or accepted, by the checks in Python as they stand."""
import numpy as np
import pytest
import torch

from paper_2601_02360_amd import binding as B

X, U, OUT = torch.zeros(8, 16), torch.zeros(16, 4), torch.zeros(8, 4)


@pytest.mark.parametrize("args", [(X, U, OUT, None, None, None, 0, None), (X, U, OUT), (), (X.numpy(), U, OUT, None, None, None, 0, None),
                                  (X, U, OUT, None, None, None, "0", None), (X[:, ::2], U, OUT, None, None, None, 0, 0),
                                  (X, U.to_sparse(), OUT, None, None, None, 0, None), (X, U, OUT, None, None, None, 0, 1 << 70)])
def test_arguments_that_are_not_plainly_right_are_handed_back(args):
    native = B._native()
    assert native.project(*args) is None and native.reconstruct(*args) is None and native.reproject(*args) is None
    assert native.compress(*args) is None and native.aggregate(*args) is None and native.outer_update(*args) is None
    assert native.aggregate_update(*args) is None and native.outer_step_batch(*args) is None


def test_null_handles_are_refused_by_the_library():
    native = B._native()
    assert native.aggregate(None, None, None, 0) == B.SPLC_EINVAL
    assert native.outer_update(None, None, None, 1.0, 0) == B.SPLC_EINVAL
    assert native.aggregate_update(None, None, None, 1.0, None, None, 0) == B.SPLC_EINVAL
    assert native.outer_step_batch(None, 1, None, None, None, 0.9, 1.0, None, None, 0, 0) == B.SPLC_EINVAL
    assert native.outer_update(None, None, None, np.float32(1.0), 0) is None            # Python converts it
    assert native.outer_step_batch(None, 1 << 40, None, None, None, 0.9, 1.0, None, None, 0, 0) is None


@pytest.mark.gpu
def test_every_form_of_argument_gives_the_same_step():
    n = 3 * 4096 + 7
    g = torch.Generator(device="cuda").manual_seed(1)
    th0, tl, ef0 = (torch.randn(n, generator=g, device="cuda") for _ in range(3))
    side = torch.cuda.Stream()
    results = []
    for beta, stream, lists in ((0.95, None, False), (np.float64(0.95), None, False), (0.95, side, False),
                                (torch.tensor(0.95, dtype=torch.float64), side.cuda_stream, False), (0.95, None, True)):
        plan = B.Plan([n], 32)
        th, ef = th0.clone(), ef0.clone()
        pairs, aux = plan.message_buffers()
        torch.cuda.synchronize()
        h = (lambda t: [t]) if lists else (lambda t: plan.bind([t], stream=stream))
        B.sparseloco_compress(plan, h(ef), pairs, aux, beta, theta_outer=h(th), theta_local=h(tl), stream=stream)
        m = plan.bind_messages([pairs], [aux], stream=stream)
        B.sparseloco_aggregate_update(plan, m, h(th), 1.0, stream=stream)
        torch.cuda.synchronize()
        results.append((th, ef, pairs, aux))
    for r in results[1:]:
        assert all(torch.equal(a, b) for a, b in zip(r, results[0]))


@pytest.mark.gpu
def test_plain_calls_are_taken(monkeypatch):
    """Every call with plain arguments is made by the native function, with status OK, and not handed back to Python."""
    native, made = B._native(), []

    class Recorded:
        def __getattr__(self, name):
            def call(*args):
                made.append((name, getattr(native, name)(*args)))
                return made[-1][1]
            return call
    monkeypatch.setattr(B, "_native", lambda: Recorded())
    n = 2 * 4096 + 5
    plan = B.Plan([n], 32)
    th, tl, ef, mean = (torch.zeros(n, device="cuda") for _ in range(4))
    hth, htl, hef, hmean = (plan.bind([t]) for t in (th, tl, ef, mean))
    delta = plan.bind([torch.zeros(n, device="cuda", dtype=torch.bfloat16)], dtype=torch.bfloat16)
    pairs, aux = plan.message_buffers()
    m = plan.bind_messages([pairs], [aux])
    x, u, out = torch.zeros(8, 16, device="cuda"), torch.zeros(16, 4, device="cuda"), torch.zeros(8, 4, device="cuda")
    table = torch.nn.Parameter(torch.zeros(5, 16, device="cuda"))
    tables = dict(t_perp=table, token_ids=torch.zeros(8, dtype=torch.int32, device="cuda"), pos_embed=torch.zeros(4, 16, device="cuda"))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for stream in (None, side, side.cuda_stream):
        made.clear()
        B.sparseloco_compress(plan, hef, pairs, aux, 0.95, theta_outer=hth, theta_local=htl, stream=stream)
        B.sparseloco_compress(plan, hef, pairs, aux, 0.95, delta=delta, stream=stream)
        B.sparseloco_aggregate(plan, m, hmean, stream=stream)
        B.sparseloco_outer_update(plan, hth, hmean, 1.0, stream=stream)
        B.sparseloco_aggregate_update(plan, m, hth, 1.0, stream=stream)
        B.sparseloco_outer_step_batch(plan, hth, htl, hef, m, 0.95, 1.0, reset=True, stream=stream)
        B.sparseloco_subspace_project(x, u, out, stream=stream)
        B.sparseloco_subspace_project(x, u, out, **tables, stream=stream)
        B.sparseloco_subspace_reconstruct(out, u, x, **tables, matmul=B.SPLC_MATMUL_BF16X3, stream=stream)
        B.sparseloco_reproject_embedding(x, torch.zeros_like(x), u, out, stream=stream)
        torch.cuda.synchronize()
        assert made == [(name, B.SPLC_OK) for name in ("compress", "compress", "aggregate", "outer_update", "aggregate_update",
                                                       "outer_step_batch", "project", "project", "reconstruct", "reproject")]


@pytest.mark.gpu
def test_what_was_refused_is_refused_with_its_reason():
    n = 4096
    plan = B.Plan([n], 32)
    th, tl, ef = (torch.zeros(n, device="cuda") for _ in range(3))
    pairs, aux = plan.message_buffers()
    hth, htl, hef = plan.bind([th]), plan.bind([tl]), plan.bind([ef])
    args = dict(theta_outer=hth, theta_local=htl)
    with pytest.raises(ValueError, match="pairs_out: 31 elements"):
        B.sparseloco_compress(plan, hef, pairs[:31], aux, 0.95, **args)
    with pytest.raises(ValueError, match="aux_out: not on a GPU"):
        B.sparseloco_compress(plan, hef, pairs, aux.cpu(), 0.95, **args)
    with pytest.raises(B.SparseLoCoError) as e:
        B.sparseloco_compress(plan, hef, pairs, aux, float("nan"), **args)
    assert e.value.status == B.SPLC_EINVAL
    other = B.Plan([n, n], 32)
    with pytest.raises(B.SparseLoCoError) as e:
        B.sparseloco_outer_update(other, hth, htl, 1.0)
    assert e.value.status == B.SPLC_EPLAN
    x, u, out = torch.zeros(8, 16, device="cuda"), torch.zeros(16, 4, device="cuda"), torch.zeros(8, 4, device="cuda")
    with pytest.raises(ValueError, match="activations"):
        B.sparseloco_subspace_project(x.double(), u, out)
    with pytest.raises(ValueError, match="contiguous"):
        B.sparseloco_subspace_project(torch.zeros(16, 8, device="cuda").t(), u, out)
    with pytest.raises(ValueError, match="token_ids"):
        B.sparseloco_subspace_project(x, u, out, t_perp=x, token_ids=torch.zeros(8, dtype=torch.int64, device="cuda"))
    with pytest.raises(ValueError, match="not on a GPU"):
        B.sparseloco_subspace_reconstruct(out, u.cpu(), x)
    with pytest.raises(B.SparseLoCoError) as e:
        B.sparseloco_subspace_project(x, u, out, matmul=7)
    assert e.value.status == B.SPLC_EINVAL
    B.sparseloco_subspace_project(torch.nn.Parameter(x), u, out)

"""Lists around a window of the order in which workgroups take their chunks (1024 groups of four): one group less, one
window, a group and a part of one more, two windows and more; full chunks, and every second one partial (then the groups
are turned).  Every kernel that walks the list, against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunks", [4092, 4096, 4099, 8192 + 2])
@pytest.mark.parametrize("partial", [False, True])
def test_work_order(oracle, chunks, partial):
    from paper_2508_15706_amd import binding as sl
    k, R, beta, lr = 16, 2, 0.95, 0.8
    descs = [(64 * (chunks // 2), 67, 0, 1)] if partial else [(1, 4096 * chunks, 0, 0)]
    n = descs[0][0] * descs[0][1]
    gen = torch.Generator(device="cuda").manual_seed(chunks + partial)
    new = lambda s: torch.empty(n, device="cuda").normal_(0, s, generator=gen)  # noqa: E731
    host = lambda x: x.cpu().numpy()  # noqa: E731
    same = lambda got, want, what: np.testing.assert_array_equal(host(got).view(np.uint32), want.view(np.uint32), what)  # noqa: E731
    plan = sl.sl_plan_create(descs, k)
    ws = sl.alloc_workspace(plan)
    pays, refs, wires, sizes = [], [], [], []
    for r in range(R):
        e, d = new(1e-3), new(1e-3)
        e_ref = host(e)
        pay, wire = sl.alloc_payload(plan), sl.alloc_coded(plan)
        sl.sl_compress_coded(plan, e, d, beta, pay, wire, ws)
        refs.append(oracle.compress(descs, k, e_ref, host(d), beta))
        assert np.array_equal(host(pay)[:plan.payload_bytes], refs[-1])
        same(e, e_ref, "e")
        pays.append(pay)
        wires.append(wire)
        sizes.append(sl.coded_size(wire))
    theta0, m0, d = new(0.02), new(1e-3), new(1e-3)
    want = host(theta0)
    oracle.decompress_avg_apply(descs, k, want, refs, lr)
    theta = theta0.clone()
    sl.sl_decompress_avg_apply(plan, theta, pays, lr)
    same(theta, want, "plain aggregate")
    theta.copy_(theta0)
    sl.sl_decompress_avg_apply_coded(plan, theta, wires, sizes, lr)
    same(theta, want, "coded aggregate")
    m, direction = m0.clone(), torch.empty_like(m0)
    sl.sl_lom_direction(plan, m, d, 0.9, direction)
    m_ref = host(m0)
    dir_ref = oracle.lom_direction(descs, m_ref, host(d), 0.9, out=np.zeros(n, np.float32))
    same(m, m_ref, "m")
    same(direction, dir_ref, "dir")
    theta.copy_(theta0)
    want = host(theta0)
    sl.sl_dense_avg_apply(plan, theta, m, [d, direction], lr, 0.9)
    oracle.dense_avg_apply(descs, want, [host(d), dir_ref], lr, m=m_ref, mu=0.9)
    same(theta, want, "dense aggregate")
    same(m, m_ref, "momentum")
    sl.sl_sub_topk(plan, m)
    oracle.sub_topk(descs, k, m_ref)
    same(m, m_ref, "Sub-k")


@pytest.mark.parametrize("chunks", [5119, 5120])
@pytest.mark.parametrize("momentum", [False, True])
def test_dense_average_lengths(oracle, chunks, momentum):
    """Both sides of the length below which the dense average requests a worker's loads together."""
    from paper_2508_15706_amd import binding as sl
    descs, n = [(64 * chunks, 64, 0, 1)], 4096 * chunks
    gen = torch.Generator(device="cuda").manual_seed(chunks)
    theta, m, a, b, c = (torch.empty(n, device="cuda").normal_(0, 1e-2, generator=gen) for _ in range(5))
    want, m_ref = theta.cpu().numpy(), m.cpu().numpy() if momentum else None
    sl.sl_dense_avg_apply(sl.sl_plan_create(descs, 8), theta, m if momentum else None, [a, b, c], 0.7, 0.9)
    oracle.dense_avg_apply(descs, want, [x.cpu().numpy() for x in (a, b, c)], 0.7, m=m_ref, mu=0.9)
    assert np.array_equal(theta.cpu().numpy().view(np.uint32), want.view(np.uint32))
    if momentum:
        assert np.array_equal(m.cpu().numpy().view(np.uint32), m_ref.view(np.uint32))

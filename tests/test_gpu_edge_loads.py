"""Matrices whose last tile column cuts through a lane's four columns, down to a single column, and runs with odd tails - at the very
start of an arena without a spare element behind it, and inside one: every kernel that reads theta, the momentum or m of a
partial chunk with whole accesses, against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 1), (70, 1), (2, 2), (67, 2), (66, 3), (64, 5), (130, 66), (3, 67), (64, 130), (5, 199), (66, 64), (1, 4096 + 5), (1, 8191)])
@pytest.mark.parametrize("inside", [False, True])
def test_edge_loads(oracle, shape, inside):
    from paper_2508_15706_amd import binding as sl
    k, layout = 4, 0 if shape[0] == 1 else 1
    descs = [(1, 64, 0, 0)] if inside else []
    off = 64 if inside else 0
    descs.append((*shape, off, layout))
    n = off + shape[0] * shape[1]
    rng = np.random.default_rng(shape[0] * 1000 + shape[1])
    new = lambda s: rng.normal(0, s, n).astype(np.float32)  # noqa: E731
    dev = lambda x: torch.from_numpy(x.copy()).cuda()  # noqa: E731
    same = lambda got, want, what: np.testing.assert_array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32), what)  # noqa: E731
    plan = sl.sl_plan_create(descs, k)
    ws = sl.alloc_workspace(plan)
    pays, wires, sizes, refs = [], [], [], []
    for _ in range(2):
        e, d = new(1e-3), new(1e-3)
        e_dev, pay, wire = dev(e), sl.alloc_payload(plan), sl.alloc_coded(plan)
        sl.sl_compress_coded(plan, e_dev, dev(d), 0.95, pay, wire, ws)
        refs.append(oracle.compress(descs, k, e, d, 0.95))
        same(e_dev, e, "e")
        assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), refs[-1])
        pays.append(pay), wires.append(wire), sizes.append(sl.coded_size(wire))
    theta0, m0, d = new(0.02), new(1e-3), new(1e-3)
    want, m_want = theta0.copy(), m0.copy()
    oracle.decompress_avg_apply(descs, k, want, refs, 0.8)
    for coded in (False, True):
        theta = dev(theta0)
        if coded:
            sl.sl_decompress_avg_apply_coded(plan, theta, wires, sizes, 0.8)
        else:
            sl.sl_decompress_avg_apply(plan, theta, pays, 0.8)
        same(theta, want, "theta")
    want = theta0.copy()
    oracle.decompress_avg_apply_nesterov_b(descs, k, 2, want, m_want, refs, 0.8, 0.9)
    for coded in (False, True):
        theta, m = dev(theta0), dev(m0)
        if coded:
            sl.sl_decompress_avg_apply_nesterov_coded(plan, theta, m, wires, sizes, 0.8, 0.9)
        else:
            sl.sl_decompress_avg_apply_nesterov(plan, theta, m, pays, 0.8, 0.9)
        same(theta, want, "theta with momentum")
        same(m, m_want, "momentum")
    m, direction, m_want = dev(m0), torch.zeros(n, device="cuda"), m0.copy()
    dir_want = oracle.lom_direction(descs, m_want, d, 0.9, out=np.zeros(n, np.float32))
    sl.sl_lom_direction(plan, m, dev(d), 0.9, direction)
    same(m, m_want, "m")
    same(direction, dir_want, "dir")
    sl.sl_sub_topk(plan, m)
    oracle.sub_topk(descs, k, m_want)
    same(m, m_want, "Sub-k")

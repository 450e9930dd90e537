"""Partial chunks - rows that end at every place inside a lane's four columns, narrow matrices with few lanes
that hold elements (the selection's bound is then poor), run tails of many lengths,
all-zero chunks - on short lists, which take several waves per chunk (test_gpu_wave_per_chunk.py has the other form), against the oracle: compress (eager, deferred, from
parameters), Sub-k and the plain aggregate with and without momentum."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = ([(80, c, 1) for c in (1, 2, 3, 4, 5, 6, 7, 8, 61, 62, 63, 65, 66, 67, 129, 134)]
          + [(129, 64, 1), (66, 64, 1)] + [(1, 4096 + t, 0) for t in (16, 17, 18, 19, 63, 65, 66, 67, 130, 4095)] + [(1, 17, 0), (1, 67, 0)])


def lists():
    descs, off = [], 0
    for r, c, lay in SHAPES:
        descs.append((r, c, off, lay))
        off += (r * c + 63) // 64 * 64
    return descs, off


@pytest.mark.parametrize("k", [4, 8, 16])
@pytest.mark.parametrize("zero", [False, True])
def test_partial_chunks(oracle, k, zero):
    from paper_2508_15706_amd import binding as sl
    descs, n = lists()
    rng = np.random.default_rng(k + zero)
    plan = sl.sl_plan_create(descs, k)
    ws = sl.alloc_workspace(plan)
    e0, d0, to, m0, theta0 = (rng.normal(0, s, n).astype(np.float32) for s in (1e-3, 1e-3, 0.02, 1e-3, 0.02))
    if zero:                                     # whole chunks of zeros, both signs, partial ones among them
        e0[:] = 0.0
        d0[::2], d0[1::2] = 0.0, -0.0
    cuda = lambda x: torch.from_numpy(x.copy()).cuda()  # noqa: E731
    same = lambda got, want, what: np.testing.assert_array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32), what)  # noqa: E731
    # eager, then a deferred round on the same state, then the pending update
    e, pay, pay2 = cuda(e0), sl.alloc_payload(plan), sl.alloc_payload(plan)
    sl.sl_compress(plan, e, cuda(d0), 0.95, pay, ws)
    e_ref = e0.copy()
    ref = oracle.compress(descs, k, e_ref, d0, 0.95)
    torch.cuda.synchronize()
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), ref)
    same(e, e_ref, "eager")
    e = cuda(e0)
    sl.sl_compress(plan, e, cuda(d0), 0.95, pay, ws, flags=sl.SL_COMPRESS_DEFER_RESIDUAL)
    sl.sl_compress(plan, e, cuda(d0), 0.95, pay2, ws, flags=sl.SL_COMPRESS_DEFER_RESIDUAL, pending=pay)
    sl.sl_residual_apply(plan, e, pay2)
    ref2 = oracle.compress(descs, k, e_ref, d0, 0.95)
    torch.cuda.synchronize()
    assert np.array_equal(pay2[:plan.payload_bytes].cpu().numpy(), ref2)
    same(e, e_ref, "deferred")
    # from parameters
    tl = (to - d0).astype(np.float32)
    e, e_ref = cuda(e0), e0.copy()
    sl.sl_compress_params(plan, e, cuda(to), cuda(tl), 0.95, pay, ws)
    refp = oracle.compress(descs, k, e_ref, (to - tl).astype(np.float32), 0.95)
    torch.cuda.synchronize()
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), refp)
    same(e, e_ref, "params")
    # Sub-k
    m, m_ref = cuda(d0 if zero else m0), (d0 if zero else m0).copy()
    sl.sl_sub_topk(plan, m)
    oracle.sub_topk(descs, k, m_ref)
    torch.cuda.synchronize()
    same(m, m_ref, "sub-k")
    # aggregates
    theta, want = cuda(theta0), theta0.copy()
    sl.sl_decompress_avg_apply(plan, theta, [pay, pay2], 0.7)
    oracle.decompress_avg_apply(descs, k, want, [refp, ref2], 0.7)
    torch.cuda.synchronize()
    same(theta, want, "theta")
    theta, mom, want, mom_ref = cuda(theta0), cuda(m0), theta0.copy(), m0.copy()
    sl.sl_decompress_avg_apply_nesterov(plan, theta, mom, [pay, pay2], 0.7, 0.9)
    oracle.decompress_avg_apply_nesterov_b(descs, k, 2, want, mom_ref, [refp, ref2], 0.7, 0.9)
    torch.cuda.synchronize()
    same(theta, want, "theta with momentum")
    same(mom, mom_ref, "momentum")


@pytest.mark.parametrize("k", [4, 12, 32, 48, 64, 100, 128, 200, 256, 300, 512])
def test_pruning_groups_of_partial_chunks(oracle, k):
    """Widths and tail lengths around the numbers of maxima that bound the threshold of a partial chunk: as many lanes with elements as
    give just under and just over 3k/2 maxima, one element per group, fewer elements than 16 groups per lane can spread."""
    from paper_2508_15706_amd import binding as sl
    descs, off = [], 0
    shapes = [(r, c, 1) for r in (64, 66, 67, 80, 96, 192) for c in (4, 8, 12, 20, 24, 28, 36, 44, 52, 60, 63, 100)]
    shapes += [(1, 4096 + t, 0) for t in (64, 100, 128, 192, 255, 256, 300, 320, 512, 513, 600, 1024, 1100, 2048, 4000)]
    for r, c, lay in shapes:
        smallest = (r * c % 4096 or 4096) if lay == 0 else (r % 64 or 64) * (c % 64 or 64)
        if smallest < k:
            continue
        descs.append((r, c, off, lay))
        off += (r * c + 63) // 64 * 64
    rng = np.random.default_rng(31 * k)
    plan = sl.sl_plan_create(descs, k)
    e0, d0 = rng.normal(0, 1e-3, off).astype(np.float32), (1e-3 * rng.standard_t(3, off)).astype(np.float32)
    e, pay = torch.from_numpy(e0.copy()).cuda(), sl.alloc_payload(plan)
    sl.sl_compress(plan, e, torch.from_numpy(d0).cuda(), 0.95, pay, sl.alloc_workspace(plan))
    e_ref = e0.copy()
    ref = oracle.compress(descs, k, e_ref, d0, 0.95)
    m, m_ref = torch.from_numpy(d0.copy()).cuda(), d0.copy()
    sl.sl_sub_topk(plan, m)
    oracle.sub_topk(descs, k, m_ref)
    torch.cuda.synchronize()
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), ref)
    assert np.array_equal(e.cpu().numpy().view(np.uint32), e_ref.view(np.uint32))
    assert np.array_equal(m.cpu().numpy().view(np.uint32), m_ref.view(np.uint32))

"""Selections of more than 512 of a chunk's elements, whose threshold is bracketed by a sample on lists of 3328 chunks and more, and with several
waves per chunk on short ones: values for which the bracket holds,
misses (elements outside the sample's registers differ from those in it) or overflows (uneven columns, ties), partial chunks, the first and the last densities.
Top-k removed in place and the payload, against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def chunk_values(rng, n_chunks):
    x = rng.normal(0, 1e-3, (n_chunks, 4096)).astype(np.float32)
    x[1] = 1e-3 * rng.standard_t(3, 4096)
    x[2, np.arange(4096) % 64 < 4] *= 50                # hot columns: one lane in sixteen holds most of the large ones
    x[3] = rng.integers(-3, 4, 4096)                    # ties
    x[4] = 0.5                                          # one value
    x[5] = 0
    x[6, rng.permutation(4096)[:700]] = 0
    r = np.arange(4096)
    sampled = (4 * (r // 256) + r % 4) % 9 == 0         # the registers that the sample takes
    x[7, sampled] *= 100                                # ... larger than all others, and smaller
    x[8, sampled] *= 0.01
    x[9] = np.float32(1e-42) * rng.integers(0, 50, 4096)        # denormal
    x[10, :8] = [3e38, -3e38, 1e30, 2, -0.0, 1e-45, 3e38, 7]
    x[11] *= np.repeat(10.0 ** rng.uniform(-6, 2, 64), 64)      # rows of any scale
    return x.astype(np.float32)


@pytest.mark.parametrize("k", [516, 520, 640, 1024, 1416, 1424, 2048, 3000, 4000, 4032, 4052, 4096])
def test_sampled_selection(oracle, k):
    from paper_2508_15706_amd import binding as sl
    rng = np.random.default_rng(k)
    x = chunk_values(rng, 13).reshape(-1)
    tail = min(4095, k + 37)                            # a partial chunk that holds little more than k
    descs = [(1, x.size, 0, 0)]
    if k < 4096:
        descs.append((1, tail, x.size, 0))
        x = np.concatenate([x, rng.normal(0, 1e-3, tail).astype(np.float32)])
    x = np.concatenate([x, np.zeros(-x.size % 64, np.float32)])
    plan = sl.sl_plan_create(descs, k)
    m = torch.from_numpy(x).cuda()
    sl.sl_sub_topk(plan, m)
    want = x.copy()
    oracle.sub_topk(descs, k, want)
    assert np.array_equal(m.cpu().numpy().view(np.uint32), want.view(np.uint32))
    e, e_ref, pay = torch.zeros(x.size, device="cuda"), np.zeros_like(x), sl.alloc_payload(plan)
    sl.sl_compress(plan, e, torch.from_numpy(x).cuda(), 0.95, pay, sl.alloc_workspace(plan))
    ref = oracle.compress(descs, k, e_ref, x, 0.95)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), ref)
    assert np.array_equal(e.cpu().numpy().view(np.uint32), e_ref.view(np.uint32))


def non_finite_values(rng):
    """Nine chunks with infinities and NaNs of every payload (the largest keys, up to one below 2^31 - 1), as words."""
    x = rng.normal(0, 1e-3, (9, 4096)).astype(np.float32).view(np.uint32)
    r = np.arange(4096)
    sampled = (4 * (r // 256) + r % 4) % 9 == 0
    payload = lambda n, low: (rng.integers(low, 0x7FFFFFFF, n) | rng.integers(0, 2, n) << 31).astype(np.uint32)  # noqa: E731
    x[0, rng.permutation(4096)[:60]] = 0x7F800000       # infinity
    x[1, rng.permutation(4096)[:60]] = 0x7FC00000       # the usual NaN
    x[2, rng.permutation(4096)[:300]] = payload(300, 0x7F800001)
    x[3] = 0
    x[3, sampled] = payload(sampled.sum(), 0x7FE00001)  # the sample's registers NaN, all others zero
    x[4, sampled] = 0
    x[4, ~sampled] = payload((~sampled).sum(), 0x7FE00001)
    x[5] = 0x7FFFFFFE
    x[6, :2100] = 0xFF800000
    x[7] = payload(4096, 0x7F800001)
    x[8, 100:160] = 0x7FFFFFFF
    return x


@pytest.mark.parametrize("k", [520, 1024, 2048, 4000])
def test_sampled_selection_non_finite(oracle, k):
    """Chunks that hold infinities and NaNs are selected by the bits of their elements like any other."""
    from paper_2508_15706_amd import binding as sl
    x = non_finite_values(np.random.default_rng(k)).reshape(-1)
    descs = [(1, x.size, 0, 0)]
    m = torch.from_numpy(x.view(np.float32).copy()).cuda()
    sl.sl_sub_topk(sl.sl_plan_create(descs, k), m)
    at = oracle.sub_topk(descs, k, x.view(np.float32).copy(), want_idx=True).reshape(9, k).astype(np.int64)
    want = x.copy()
    want[(4096 * np.arange(9)[:, None] + at).reshape(-1)] = 0
    assert np.array_equal(m.cpu().numpy().view(np.uint32), want)


@pytest.mark.parametrize("k, chunks", [(516, 3328), (520, 3327), (520, 3328), (640, 3328), (1024, 3328), (1416, 3328), (1424, 3328), (2048, 3328),
                                       (3000, 3328), (4000, 3328), (4032, 3328), (4052, 3328)])
def test_sampled_selection_long_lists(oracle, k, chunks):
    """The length from which the sample is used: the chunks of the tests above among others of normal values."""
    from paper_2508_15706_amd import binding as sl
    rng = np.random.default_rng(k)
    odd = np.concatenate([chunk_values(rng, 13), non_finite_values(rng).view(np.float32)])
    x = np.concatenate([odd, np.tile(rng.normal(0, 1e-3, (61, 4096)).astype(np.float32), (60, 1))])[:chunks]
    descs, n = [(1, x.size, 0, 0)], x.size
    plan = sl.sl_plan_create(descs, k)
    m = torch.from_numpy(x.reshape(-1).copy()).cuda()
    sl.sl_sub_topk(plan, m)
    at = oracle.sub_topk(descs, k, x.reshape(-1).copy(), want_idx=True).reshape(chunks, k).astype(np.int64)
    want = x.reshape(-1).view(np.uint32).copy()
    want[(4096 * np.arange(chunks)[:, None] + at).reshape(-1)] = 0
    assert np.array_equal(m.cpu().numpy().view(np.uint32), want)
    x[13:22] = x[22:31]                                  # (a NaN's payload is not part of what a sum promises)
    x = x.reshape(-1)
    e, e_ref, pay = torch.zeros(n, device="cuda"), np.zeros_like(x), sl.alloc_payload(plan)
    sl.sl_compress(plan, e, torch.from_numpy(x).cuda(), 0.95, pay, sl.alloc_workspace(plan))
    ref = oracle.compress(descs, k, e_ref, x, 0.95)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), ref)
    assert np.array_equal(e.cpu().numpy().view(np.uint32), e_ref.view(np.uint32))

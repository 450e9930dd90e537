"""Aggregates with several waves on one chunk (short lists, few workers) and with one: list lengths, worker counts and densities
on both sides of every place where the number of waves changes, with partial chunks and clustered supports; plain and
coded payloads, with and without the global momentum, against the oracle.  And plain records whose indices do not ascend."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (k, value bits, chunks, workers)
CASES = [(64, 2, 256, 8), (64, 2, 257, 8), (64, 2, 257, 4), (128, 4, 256, 5), (136, 2, 512, 8), (256, 2, 513, 8), (264, 2, 100, 3), (32, 1, 1024, 4),
         (32, 1, 1025, 3), (8, 3, 1281, 8), (16, 2, 2048, 2), (64, 32, 300, 4), (128, 32, 40, 8), (4, 2, 200, 1), (100, 2, 700, 9), (256, 2, 60, 4), (72, 4, 30, 4), (32, 32, 100, 9), (64, 4, 40, 17)]


@pytest.mark.parametrize("k, bits, chunks, R", CASES)
@pytest.mark.parametrize("ragged", [False, True])
def test_both_forms(oracle, k, bits, chunks, R, ragged):
    from paper_2508_15706_amd import binding as sl
    shapes = [(130, 67, 1), (200, 530, 1), (1, 4096 + 700, 0), (66, 64, 1)]
    fits = lambda r, c, lay: (r * c % 4096 or 4096) >= k if lay == 0 else (r % 64 or 64) * (c % 64 or 64) >= k  # noqa: E731
    count = lambda r, c, lay: -(-r * c // 4096) if lay == 0 else -(-r // 64) * -(-c // 64)  # noqa: E731
    shapes = [s for s in shapes if ragged and fits(*s)]
    while sum(count(*s) for s in shapes) >= chunks:
        shapes.pop()
    shapes.append((64 * (chunks - sum(count(*s) for s in shapes)), 64, 1))
    descs, n = [], 0
    for r, c, lay in shapes:
        descs.append((r, c, n, lay))
        n += (r * c + 63) // 64 * 64
    rng = np.random.default_rng(k + chunks + R)
    plan = sl.sl_plan_create_bits(descs, k, bits)
    assert plan.num_chunks == chunks
    theta0, m0 = rng.normal(0, 0.02, n).astype(np.float32), rng.normal(0, 1e-3, n).astype(np.float32)
    pays, coded = [], []
    for r in range(R):
        x = rng.normal(0, 1e-3, n).astype(np.float32)
        if r % 3 == 1:                           # one cluster per chunk: all selected entries in one wave's part, or across a border
            x.reshape(-1, 64)[5::64] *= 1000
        pays.append(oracle.compress_b(descs, k, bits, x.copy(), x, 0.0, ef_frozen=True))
        coded.append(oracle.rice_encode_b(descs, k, bits, pays[-1]))
    cuda = lambda x: torch.from_numpy(x.copy()).cuda()  # noqa: E731
    same = lambda got, want: np.testing.assert_array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32))  # noqa: E731
    want, want_n, want_m = theta0.copy(), theta0.copy(), m0.copy()
    oracle.decompress_avg_apply_b(descs, k, bits, want, pays, 0.8)
    oracle.decompress_avg_apply_nesterov_b(descs, k, bits, want_n, want_m, pays, 0.8, 0.9)
    gp, gc = [cuda(p) for p in pays], [cuda(p) for p in coded]
    sizes = [p.size for p in coded]
    t = cuda(theta0)
    sl.sl_decompress_avg_apply(plan, t, gp, 0.8)
    same(t, want)
    t = cuda(theta0)
    sl.sl_decompress_avg_apply_coded(plan, t, gc, sizes, 0.8)
    same(t, want)
    t, m = cuda(theta0), cuda(m0)
    sl.sl_decompress_avg_apply_nesterov(plan, t, m, gp, 0.8, 0.9)
    same(t, want_n), same(m, want_m)
    t, m = cuda(theta0), cuda(m0)
    sl.sl_decompress_avg_apply_nesterov_coded(plan, t, m, gc, sizes, 0.8, 0.9)
    same(t, want_n), same(m, want_m)


@pytest.mark.parametrize("k, chunks", [(64, 20), (128, 600), (256, 20)])
def test_indices_in_any_order(oracle, k, chunks):
    from paper_2508_15706_amd import binding as sl
    descs, n, R = [(64 * chunks, 64, 0, 1)], 4096 * chunks, 3
    rng = np.random.default_rng(k)
    plan = sl.sl_plan_create(descs, k)
    pays = []
    for r in range(R):
        idx = np.argsort(rng.random((chunks, 4096)), axis=1)[:, :k].astype(np.uint16)
        out = torch.zeros(chunks * 7 * k // 4, dtype=torch.uint8, device="cuda")
        sl.sl_pack_indices(torch.from_numpy(idx.reshape(-1).copy()).cuda(), torch.from_numpy(rng.integers(0, 4, chunks * k, dtype=np.uint8)).cuda(), chunks, k, out)
        pay = np.zeros(plan.payload_bytes, np.uint8)
        pay[:16] = rng.normal(0, 1e-3, 4).astype(np.float32).view(np.uint8)
        pay[16:16 + out.numel()] = out.cpu().numpy()
        pays.append(pay)
    want = rng.normal(0, 0.02, n).astype(np.float32)
    t = torch.from_numpy(want.copy()).cuda()
    oracle.decompress_avg_apply(descs, k, want, pays, 0.7)
    sl.sl_decompress_avg_apply(plan, t, [torch.from_numpy(p).cuda() for p in pays], 0.7)
    np.testing.assert_array_equal(t.cpu().numpy().view(np.uint32), want.view(np.uint32))

"""Selection with several waves on one chunk (short lists) and with one: list lengths on both sides of every place where the
number of waves changes, or the streaming hint comes and goes with the eager update, with partial chunks - narrow tiles, run tails with fewer groups than k, more than the candidate list
holds - all-zero chunks, chunks of few distinct values (ties), clustered ones, and heavy tails.  Eager, deferred (the
record of the round before is still pending), frozen, from parameters, coded, and Sub-k, against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (k, value bits, chunks of the list): 8 | 4 | 1 waves
CASES = [(32, 2, 512), (64, 2, 513), (128, 1, 6144), (64, 4, 6145), (136, 2, 512), (200, 3, 2048), (256, 2, 2049), (264, 2, 512), (512, 32, 768),
         (500, 2, 769), (64, 2, 2047), (32, 3, 2048), (136, 2, 9216), (256, 2, 9217), (520, 2, 512), (1024, 4, 3072), (2048, 2, 3073), (4, 2, 513), (4096, 2, 40), (1448, 32, 600)]


@pytest.mark.parametrize("k, bits, chunks", CASES)
def test_both_forms(oracle, k, bits, chunks):
    from paper_2508_15706_amd import binding as sl
    shapes = [(130, 67, 1), (200, 530, 1), (64, 18, 1), (1, 4096 + 700, 0), (1, 4096 + 1100, 0), (1, 2 * 4096 + 33, 0), (66, 64, 1)]
    fits = lambda r, c, lay: (r * c % 4096 or 4096) >= k if lay == 0 else (r % 64 or 64) * (c % 64 or 64) >= k  # noqa: E731
    count = lambda r, c, lay: -(-r * c // 4096) if lay == 0 else -(-r // 64) * -(-c // 64)  # noqa: E731
    shapes = [s for s in shapes if fits(*s)]
    rest = chunks - sum(count(*s) for s in shapes)
    shapes = [(64 * 8, 64, 1)] + shapes + [(1, 4096 * (rest - 8), 0)]
    descs, n = [], 0
    for r, c, lay in shapes:
        descs.append((r, c, n, lay))
        n += (r * c + 63) // 64 * 64
    rng = np.random.default_rng(k + chunks)
    new = lambda s: rng.normal(0, s, n).astype(np.float32)  # noqa: E731
    e0, d0, d1 = new(1e-3), (1e-3 * rng.standard_t(3, n)).astype(np.float32), new(1e-3)
    tile = lambda x, i: x[4096 * i:4096 * (i + 1)]  # noqa: E731
    for x in (e0, d0, d1):                       # the first matrix's chunks: zeros, three values, a tenth of one value, a cluster
        tile(x, 0)[:] = 0.0
        tile(x, 1)[:] = np.sign(tile(x, 1)) * np.where(rng.random(4096) < 0.5, 1e-3, 2e-3).astype(np.float32)
        tile(x, 2)[rng.random(4096) < 0.1] = 0.0
        tile(x, 3)[1000:1600] *= 100
        tile(x, 4)[:] = np.float32(1e-3)
    tile(e0, 1)[:] = 0.0
    tile(e0, 4)[:] = 0.0
    plan = sl.sl_plan_create_bits(descs, k, bits)
    assert plan.num_chunks == chunks
    ws, cuda = sl.alloc_workspace(plan), lambda x: torch.from_numpy(x.copy()).cuda()  # noqa: E731
    same = lambda got, want: np.testing.assert_array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32))  # noqa: E731
    # eager
    e, want_e, pay, out = cuda(e0), e0.copy(), sl.alloc_payload(plan), sl.alloc_coded(plan)
    want = oracle.compress_b(descs, k, bits, want_e, d0, 0.95)
    sl.sl_compress(plan, e, cuda(d0), 0.95, pay, ws)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)
    same(e, want_e)
    # deferred, then coded with the first round pending
    e, pay2 = cuda(e0), sl.alloc_payload(plan)
    sl.sl_compress(plan, e, cuda(d0), 0.95, pay, ws, flags=sl.SL_COMPRESS_DEFER_RESIDUAL)
    sl.sl_compress_coded(plan, e, cuda(d1), 0.95, pay2, out, ws, flags=sl.SL_COMPRESS_DEFER_RESIDUAL, pending=pay)
    want2 = oracle.compress_b(descs, k, bits, want_e, d1, 0.95)
    coded = oracle.rice_encode_b(descs, k, bits, want2)
    assert np.array_equal(pay2[:plan.payload_bytes].cpu().numpy(), want2)
    assert np.array_equal(out[:coded.size].cpu().numpy(), coded)
    sl.sl_residual_apply(plan, e, pay2)
    same(e, want_e)
    # frozen, and from parameters
    sl.sl_compress(plan, None, cuda(d1), 0.95, pay, ws, flags=sl.SL_COMPRESS_EF_FROZEN)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), oracle.compress_b(descs, k, bits, e0.copy(), d1, 0.95, ef_frozen=True))
    outer = new(0.02)
    local = outer - d1
    e, want_e = cuda(e0), e0.copy()
    sl.sl_compress_params(plan, e, cuda(outer), cuda(local), 0.95, pay, ws)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), oracle.compress_b(descs, k, bits, want_e, outer - local, 0.95))
    same(e, want_e)
    # Sub-k
    m, want_m = cuda(d0), d0.copy()
    sl.sl_sub_topk(plan, m)
    oracle.sub_topk(descs, k, want_m)
    same(m, want_m)


@pytest.mark.parametrize("k, chunks", [(64, 500), (1500, 40), (256, 600), (1500, 600)])
def test_ties_without_number(oracle, k, chunks):
    """More keys than the list of candidates holds share the threshold, or the lower end of the bracket is not the threshold."""
    from paper_2508_15706_amd import binding as sl
    rng, n = np.random.default_rng(k), 4096 * chunks
    x = rng.normal(0, 1e-3, (chunks, 4096)).astype(np.float32)
    sign = np.where(rng.random((7, 4096)) < 0.5, -1, 1).astype(np.float32)
    x[0] = 0.0
    x[0, rng.permutation(4096)[:8]] = 1e-3       # few values among zeros
    x[1] = np.float32(1e-3) * sign[1]            # one magnitude
    x[2] = 0.0
    order = rng.permutation(4096)
    x[2, order[:3000]], x[2, order[:k + 10]] = 1e-3, 2e-3    # the upper level holds a few more than k
    x[2] *= sign[2]
    x[3] = 0.0
    # exactly k keys of one magnitude, the sample's positions (those of eight waves) all among them
    wave, lane = np.divmod(np.arange(512), 64)
    sample = 256 * (2 * wave + ((lane & 7) >> 2)) + 4 * lane + (lane & 3)
    rest = np.setdiff1d(rng.permutation(4096), sample)
    x[3, np.concatenate([sample, rest])[:k]] = 1e-3
    x[4] = 0.0
    x[5] = np.float32(3e38) * sign[5]
    x[6] = np.round(x[6] * 2e3) / 2e3            # levels
    x = x.reshape(-1)
    descs = [(64 * chunks, 64, 0, 0)]
    plan = sl.sl_plan_create(descs, k)
    ws, pay = sl.alloc_workspace(plan), sl.alloc_payload(plan)
    sl.sl_compress(plan, None, torch.from_numpy(x).cuda(), 0.95, pay, ws, flags=sl.SL_COMPRESS_EF_FROZEN)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), oracle.compress_b(descs, k, 2, np.zeros(n, np.float32), x, 0.95, ef_frozen=True))
    m, want = torch.from_numpy(x.copy()).cuda(), x.copy()
    sl.sl_sub_topk(plan, m)
    oracle.sub_topk(descs, k, want)
    np.testing.assert_array_equal(m.cpu().numpy().view(np.uint32), want.view(np.uint32))

"""The kernels that give a chunk to one wave, which short lists do not reach (sl_select_waves, sl_apply_waves): lists of narrow and cut tiles, run tails,
chunks of ties, zeros, denormals, one magnitude and clusters, followed by as many full chunks as these kernels begin at. The full chunks are one tensor
many times over, so the oracle sees it once; few of all rows are unaligned, so the accesses keep the streaming hint. Compress eager, deferred, with a pending
record, from parameters, frozen and coded; Sub-k; both aggregates with and without momentum."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FILL = 64                # chunks of the repeated tensor
SHAPES = ([(80, c, 1) for c in (1, 2, 3, 4, 5, 6, 7, 8, 61, 63, 65, 66, 67, 134)] + [(r, c, 1) for r in (64, 66, 96) for c in (12, 24, 36, 52, 100)] + [(129, 64, 1)]
          + [(1, 4096 + t, 0) for t in (16, 18, 67, 130, 255, 320, 513, 600, 1100, 2048, 4095)] + [(1, 17, 0), (1, 67, 0)])
CASES = [(4, 2), (16, 1), (16, 3), (32, 2), (32, 4), (64, 2), (64, 32), (100, 2), (128, 2), (128, 4), (136, 2), (200, 3), (256, 2), (264, 2), (512, 2), (512, 32),
         (520, 2), (1024, 4), (2048, 2)]


class List:
    """Edge tensors and the repeated one; arrays and payloads of the first repetition are the oracle's, the GPU's are whole."""

    def __init__(self, oracle, edges, k, bits):
        self.small, n = [], 0
        for r, c, lay in edges:
            self.small.append((r, c, n, lay))
            n += (r * c + 63) // 64 * 64
        self.edge = n
        first = (1, 4096 * FILL, n, 0)
        below = 6145 if k <= 128 else 2049 if k <= 256 else 769 if k <= 512 else 3073 if k < 1024 else 3329
        self.times = -(-below // FILL)
        self.whole = self.small + [(1, 4096 * FILL, n + 4096 * FILL * i, 0) for i in range(self.times)]
        self.edge_bytes = oracle.payload_bytes_b(self.small, k, bits)
        self.small.append(first)
        self.block = oracle.tensor_block_bytes_b(first, k, bits)
        self.n = n + 4096 * FILL

    def cuda(self, x):
        t = torch.from_numpy(x.copy()).cuda()
        return torch.cat([t[:self.edge], t[self.edge:].repeat(self.times)])

    def _same(self, got, want, edge):
        one = want.size - edge
        rows = got[edge:edge + self.times * one].view(self.times, one)
        assert torch.equal(rows, rows[:1].expand_as(rows))
        np.testing.assert_array_equal(got[:want.size].cpu().numpy(), want)

    def same(self, got, want):
        self._same(got.view(torch.int32), want.view(np.int32), self.edge)

    def same_payload(self, got, want):
        self._same(got, want, self.edge_bytes)


def fits(k):
    return [s for s in SHAPES if ((s[0] * s[1] % 4096 or 4096) if s[2] == 0 else (s[0] % 64 or 64) * (s[1] % 64 or 64)) >= k]


@pytest.mark.parametrize("k, bits", CASES)
def test_edges(oracle, k, bits):
    from paper_2508_15706_amd import binding as sl
    L = List(oracle, [(64 * 8, 64, 1)] + fits(k), k, bits)
    rng = np.random.default_rng(10 * k + bits)
    new = lambda s: rng.normal(0, s, L.n).astype(np.float32)  # noqa: E731
    e0, d0, d1, theta0, m0, outer = new(1e-3), (1e-3 * rng.standard_t(3, L.n)).astype(np.float32), new(1e-3), new(0.02), new(1e-3), new(0.02)
    e0[:8 * 4096] = 0.0                          # the first matrix's chunks
    x = d0[:8 * 4096].reshape(8, 4096)
    sign = np.where(rng.random(4096) < 0.5, -1, 1).astype(np.float32)
    x[0] = 0.0
    x[1] = sign * np.where(rng.random(4096) < 0.5, 1e-3, 2e-3).astype(np.float32)
    x[2, rng.random(4096) < 0.9] = 0.0
    x[3, 1000:1600] *= 100
    x[4] = np.float32(1e-3)
    x[5] = sign * rng.integers(0, 3 * k, 4096).astype(np.uint32).view(np.float32)      # denormals, some of them equal
    x[6] = np.round(x[6] * 2e3) / 2e3
    plan = sl.sl_plan_create_bits(L.whole, k, bits)
    ws, pay, pay2, pay3 = sl.alloc_workspace(plan), *(sl.alloc_payload(plan) for _ in range(3))
    out = sl.alloc_coded(plan)
    defer = sl.SL_COMPRESS_DEFER_RESIDUAL
    # eager
    e, want_e = L.cuda(e0), e0.copy()
    sl.sl_compress(plan, e, L.cuda(d0), 0.95, pay, ws)
    want = oracle.compress_b(L.small, k, bits, want_e, d0, 0.95)
    L.same_payload(pay, want), L.same(e, want_e)
    # deferred; coded with that record pending; from parameters with that one
    e = L.cuda(e0)
    sl.sl_compress(plan, e, L.cuda(d0), 0.95, pay, ws, flags=defer)
    sl.sl_compress_coded(plan, e, L.cuda(d1), 0.95, pay2, out, ws, flags=defer, pending=pay)
    want2 = oracle.compress_b(L.small, k, bits, want_e, d1, 0.95)
    L.same_payload(pay, want), L.same_payload(pay2, want2)
    size = sl.coded_size(out)
    sl.sl_rice_decode(plan, out, size, pay3)
    L.same_payload(pay3, want2)
    local = outer - d1
    sl.sl_compress_params(plan, e, L.cuda(outer), L.cuda(local), 0.95, pay3, ws, flags=defer, pending=pay2)
    want3 = oracle.compress_b(L.small, k, bits, want_e, outer - local, 0.95)
    sl.sl_residual_apply(plan, e, pay3)
    L.same_payload(pay3, want3), L.same(e, want_e)
    # frozen, Sub-k
    sl.sl_compress(plan, None, L.cuda(d0), 0.95, pay3, ws, flags=sl.SL_COMPRESS_EF_FROZEN)
    L.same_payload(pay3, oracle.compress_b(L.small, k, bits, e0.copy(), d0, 0.95, ef_frozen=True))
    m, want_m = L.cuda(d0), d0.copy()
    sl.sl_sub_topk(plan, m)
    oracle.sub_topk(L.small, k, want_m)
    L.same(m, want_m)
    # aggregates
    for R in (1, 3, 8):
        gp, wp = ([pay, pay2] * 4)[:R], ([want, want2] * 4)[:R]
        t, w = L.cuda(theta0), theta0.copy()
        sl.sl_decompress_avg_apply(plan, t, gp, 0.8)
        oracle.decompress_avg_apply_b(L.small, k, bits, w, wp, 0.8)
        L.same(t, w)
        t, m, w, wm = L.cuda(theta0), L.cuda(m0), theta0.copy(), m0.copy()
        sl.sl_decompress_avg_apply_nesterov(plan, t, m, gp, 0.8, 0.9)
        oracle.decompress_avg_apply_nesterov_b(L.small, k, bits, w, wm, wp, 0.8, 0.9)
        L.same(t, w), L.same(m, wm)
        t, m, w, wm = L.cuda(theta0), L.cuda(m0), theta0.copy(), m0.copy()
        sl.sl_decompress_avg_apply_nesterov_coded(plan, t, m, [out] * R, [size] * R, 0.8, 0.9)
        oracle.decompress_avg_apply_nesterov_b(L.small, k, bits, w, wm, [want2] * R, 0.8, 0.9)
        L.same(t, w), L.same(m, wm)
        t, w = L.cuda(theta0), theta0.copy()
        sl.sl_decompress_avg_apply_coded(plan, t, [out] * R, [size] * R, 0.8)
        oracle.decompress_avg_apply_b(L.small, k, bits, w, [want2] * R, 0.8)
        L.same(t, w)


@pytest.mark.parametrize("k", [8, 32, 64, 100, 128, 200, 300, 512, 520, 1024])
def test_non_finite(oracle, k):
    """NaNs of both signs, infinities, chunks full of either: the selected positions are the oracle's (NaN > infinity > finite as keys)."""
    from paper_2508_15706_amd import binding as sl
    edges = [(64 * 6, 64, 1)] + [s for s in fits(k) if s[1] in (7, 67, 100, 4096 + 1100)]
    L = List(oracle, edges, k, 2)
    rng = np.random.default_rng(k)
    d0 = rng.normal(0, 1e-3, L.n).astype(np.float32)
    n = L.edge
    bad = rng.choice(n, n // 20, replace=False)
    d0[bad] = rng.choice(np.array([np.nan, -np.nan, np.inf, -np.inf], np.float32), bad.size)
    d0[:4096], d0[4096:8192] = np.nan, -np.inf
    d0[8192:8192 + 4096] = np.where(rng.random(4096) < 0.5, np.float32(np.inf), d0[8192:8192 + 4096])
    plan = sl.sl_plan_create(L.whole, k)
    ws, pay = sl.alloc_workspace(plan), sl.alloc_payload(plan)
    sl.sl_compress(plan, None, L.cuda(d0), 0.95, pay, ws, flags=sl.SL_COMPRESS_EF_FROZEN)
    assert sl.sl_payload_validate(plan, pay, ws)
    want, detail = oracle.compress_b(L.small, k, 2, np.zeros(L.n, np.float32), d0, 0.95, ef_frozen=True, want_detail=True)
    got, rec, at, c = pay.cpu().numpy(), oracle.record_bytes(k), 0, 0
    for d in L.small:
        for i in range(oracle.tensor_chunks(d)):
            idx, _ = oracle.unpack_record(got[at + 16 + i * rec:at + 16 + (i + 1) * rec], k)
            assert np.array_equal(idx, detail["idx"][c * k:(c + 1) * k]), (d, i)
            c += 1
        at += oracle.tensor_block_bytes(d, k)
    assert np.array_equal(got[L.edge_bytes:at], want[L.edge_bytes:])
    m, want_m = L.cuda(d0), d0.copy()
    sl.sl_sub_topk(plan, m)
    at = oracle.sub_topk(L.small, k, d0.copy(), want_idx=True).reshape(-1, k)
    chunks = [(d, i) for d in L.small for i in range(oracle.tensor_chunks(d))]
    for (d, i), idx in zip(chunks, at):          # (+0.0 at every selected position, also where x - x is NaN)
        want_m[[oracle.element_of(d, i, int(j)) for j in idx]] = 0.0
    L.same(m, want_m)


@pytest.mark.parametrize("k, R", [(264, 3), (64, 9)])
@pytest.mark.parametrize("sizes", [[679, 1], [681], [1025, 339], [1365]])
def test_chunks_per_workgroup(oracle, k, R, sizes):
    """Aggregates of lists on both sides of where workgroups change between one chunk and four, at a density and a worker count that several
    waves per chunk do not serve."""
    from paper_2508_15706_amd import binding as sl
    descs, n = [], 0
    for c in sizes:
        descs.append((64, 64 * c, n, 1))
        n += 4096 * c
    rng = np.random.default_rng(n + k)
    plan = sl.sl_plan_create(descs, k)
    pays = [oracle.compress(descs, k, np.zeros(n, np.float32), rng.normal(0, 1e-3, n).astype(np.float32), 0.0, ef_frozen=True) for _ in range(3)]
    theta0, m0 = rng.normal(0, 0.02, n).astype(np.float32), rng.normal(0, 1e-3, n).astype(np.float32)
    cuda = lambda x: torch.from_numpy(x.copy()).cuda()  # noqa: E731
    coded = [oracle.rice_encode(descs, k, p) for p in pays]
    gp, gc, sizes_ = [cuda(p) for p in pays] * 3, [cuda(p) for p in coded] * 3, [p.size for p in coded] * 3
    same = lambda got, want: np.testing.assert_array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32))  # noqa: E731
    want, want_n, want_m = theta0.copy(), theta0.copy(), m0.copy()
    oracle.decompress_avg_apply(descs, k, want, (pays * 3)[:R], 0.8)
    oracle.decompress_avg_apply_nesterov_b(descs, k, 2, want_n, want_m, (pays * 3)[:R], 0.8, 0.9)
    t = cuda(theta0)
    sl.sl_decompress_avg_apply(plan, t, gp[:R], 0.8)
    same(t, want)
    t = cuda(theta0)
    sl.sl_decompress_avg_apply_coded(plan, t, gc[:R], sizes_[:R], 0.8)
    same(t, want)
    t, m = cuda(theta0), cuda(m0)
    sl.sl_decompress_avg_apply_nesterov(plan, t, m, gp[:R], 0.8, 0.9)
    same(t, want_n), same(m, want_m)
    t, m = cuda(theta0), cuda(m0)
    sl.sl_decompress_avg_apply_nesterov_coded(plan, t, m, gc[:R], sizes_[:R], 0.8, 0.9)
    same(t, want_n), same(m, want_m)

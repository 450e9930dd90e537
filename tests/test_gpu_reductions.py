"""Statistics, centroids and placement of the coded format at the edges of their block reductions (256,
4096 and 65536 leaves; groups of 16 chunks; several tensors) against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits, k", [(2, 8), (2, 4), (4, 8), (32, 8)])
def test_tensor_sizes_at_tile_edges(oracle, bits, k):
    from paper_2508_15706_amd import binding as sl
    # flat tensors of so many chunks, the last one cut to 8 elements: a short chunk each, so that lists with
    # many chunks stay small (runs of 4096 elements, k of them selected)
    descs, off = [], 0
    for chunks in (1, 2, 15, 16, 17, 255, 256, 257, 1023, 1025, 4095, 4097, 8193, 12289):
        n = 4096 * (chunks - 1) + 8
        descs.append((1, n, off, sl.SL_LAYOUT_FLAT))
        off += (n + 63) // 64 * 64
    g = torch.Generator(device="cuda").manual_seed(bits + k)
    delta = torch.randn(off, device="cuda", generator=g)
    plan = sl.sl_plan_create_bits(descs, k, bits)
    pay, ws = sl.alloc_payload(plan), sl.alloc_workspace(plan)
    pay.fill_(0xAB)
    coded = torch.full((sl.sl_rice_max_bytes(plan),), 0xCD, dtype=torch.uint8, device="cuda")
    e = torch.zeros(off, dtype=torch.float32, device="cuda")
    sl.sl_compress_coded(plan, e, delta, 0.95, pay, coded, ws, flags=sl.SL_COMPRESS_DEFER_RESIDUAL)
    torch.cuda.synchronize()
    want = oracle.compress_b(descs, k, bits, np.zeros(off, np.float32), delta.cpu().numpy(), 0.95)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)
    size = sl.coded_size(coded)
    assert np.array_equal(coded[:size].cpu().numpy(), oracle.rice_encode_b(descs, k, bits, want))


def test_more_than_65536_leaves(oracle):
    from paper_2508_15706_amd import binding as sl
    n = 4096 * 65601 + 100                       # 65,602 chunks of one tensor: a second round of tiles
    delta = torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(5))
    plan = sl.sl_plan_create([(1, n, 0, sl.SL_LAYOUT_FLAT)], 4)
    pay, ws = sl.alloc_payload(plan), sl.alloc_workspace(plan)
    e = torch.zeros(n, dtype=torch.float32, device="cuda")
    sl.sl_compress(plan, e, delta, 0.95, pay, ws, flags=sl.SL_COMPRESS_DEFER_RESIDUAL)
    torch.cuda.synchronize()
    want = oracle.compress([(1, n, 0, sl.SL_LAYOUT_FLAT)], 4, np.zeros(n, np.float32), delta.cpu().numpy(), 0.95)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)


@pytest.mark.parametrize("k", [352, 356, 360, 512, 1024, 2048, 4096])
def test_placement_of_long_vectors(oracle, k):
    """Vectors of 32, 33 and more words: a group's vectors are placed by (chunk, word) pairs or a chunk per turn;
    groups of 16, of 1 and of 13 chunks, supports spread and in one block (the shortest and longest vectors)."""
    from paper_2508_15706_amd import binding as sl
    descs, off = [], 0
    for chunks in (16, 33, 13):
        descs.append((1, 4096 * chunks, off, sl.SL_LAYOUT_FLAT))
        off += 4096 * chunks
    rng = np.random.default_rng(k)
    d0 = rng.normal(0, 1e-3, off).astype(np.float32)
    j = np.arange(off) % 4096
    d0[(j >= 4096 - k) & (np.arange(off) // 4096 % 3 == 1)] += 1.0             # every third chunk: the last k positions
    d0[(j < k) & (np.arange(off) // 4096 % 3 == 2)] += 1.0                       # ... and the first
    plan = sl.sl_plan_create(descs, k)
    pay, ws = sl.alloc_payload(plan), sl.alloc_workspace(plan)
    coded, again = (torch.full((sl.sl_rice_max_bytes(plan),), 0xCD, dtype=torch.uint8, device="cuda") for _ in range(2))
    e = torch.zeros(off, dtype=torch.float32, device="cuda")
    sl.sl_compress_coded(plan, e, torch.from_numpy(d0).cuda(), 0.95, pay, coded, ws)
    sl.sl_rice_encode(plan, pay, again, ws)
    torch.cuda.synchronize()
    want = oracle.compress(descs, k, np.zeros(off, np.float32), d0, 0.95)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)
    want = oracle.rice_encode(descs, k, want)
    for what, buf in (("compress", coded), ("transcoder", again)):
        size = sl.coded_size(buf)
        assert size == want.size and np.array_equal(buf[:size].cpu().numpy(), want), what


@pytest.mark.parametrize("bits, n_tensors", [(1, 550), (1, 551), (2, 412), (2, 413), (3, 275), (3, 276), (4, 165), (4, 166),
                                             (32, 512), (32, 513), (2, 1300)])
def test_lists_of_many_tensors(oracle, bits, n_tensors):
    """Both sides of the numbers of tensors where the placement steps get launches of their own and where the
    group scan goes from 1024 to 256 threads; compress and transcoder, eager error update."""
    from paper_2508_15706_amd import binding as sl
    k, descs, off = 16, [], 0
    for t in range(n_tensors):
        n = (24, 4096 + 40, 64, 2 * 4096, 100)[t % 5] if t != 7 else 4096 * 300 + 24    # 7: more groups than one turn of 16
        descs.append((1, n, off, sl.SL_LAYOUT_FLAT))
        off += (n + 63) // 64 * 64
    rng = np.random.default_rng(100 * bits + n_tensors)
    d0 = (1e-3 * rng.standard_t(3, off)).astype(np.float32)
    plan = sl.sl_plan_create_bits(descs, k, bits)
    pay, ws = sl.alloc_payload(plan), sl.alloc_workspace(plan)
    pay.fill_(0xAB)
    cap = sl.sl_rice_max_bytes(plan)
    coded, again = (torch.full((cap,), 0xCD, dtype=torch.uint8, device="cuda") for _ in range(2))
    e = torch.zeros(off, dtype=torch.float32, device="cuda")
    sl.sl_compress_coded(plan, e, torch.from_numpy(d0).cuda(), 0.95, pay, coded, ws)
    sl.sl_rice_encode(plan, pay, again, ws)
    torch.cuda.synchronize()
    e_ref = np.zeros(off, np.float32)
    want = oracle.compress_b(descs, k, bits, e_ref, d0, 0.95)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)
    assert np.array_equal(e.cpu().numpy().view(np.uint32), e_ref.view(np.uint32))
    want = oracle.rice_encode_b(descs, k, bits, want)
    for what, buf in (("compress", coded), ("transcoder", again)):
        size = sl.coded_size(buf)
        assert size == want.size and np.array_equal(buf[:size].cpu().numpy(), want), what


@pytest.mark.parametrize("bits", [1, 2, 4])
def test_pieces_of_large_tensors(oracle, bits):
    """Tensors on both sides of 10,240 chunks, from where their sums are taken in pieces of 256: the last piece full and of one
    leaf, pieces that begin at any group of the list, small tensors between."""
    from paper_2508_15706_amd import binding as sl
    descs, off, k = [], 0, 8
    for chunks in (3, 10240, 10241, 40, 10496, 1):
        descs.append((1, 4096 * chunks, off, sl.SL_LAYOUT_FLAT))
        off += 4096 * chunks
    delta = torch.randn(off, device="cuda", generator=torch.Generator(device="cuda").manual_seed(bits))
    plan = sl.sl_plan_create_bits(descs, k, bits)
    pay, coded, ws = sl.alloc_payload(plan), sl.alloc_coded(plan), sl.alloc_workspace(plan)
    sl.sl_compress_coded(plan, None, delta, 0.95, pay, coded, ws, flags=sl.SL_COMPRESS_EF_FROZEN)
    torch.cuda.synchronize()
    want = oracle.compress_b(descs, k, bits, np.zeros(off, np.float32), delta.cpu().numpy(), 0.95, ef_frozen=True)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)
    assert np.array_equal(coded[:sl.coded_size(coded)].cpu().numpy(), oracle.rice_encode_b(descs, k, bits, want))

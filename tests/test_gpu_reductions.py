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

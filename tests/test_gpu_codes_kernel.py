"""The code kernel at the edges of its mapping (eight entries per lane, 1 .. 64 lanes per chunk, then
2, 4 and 8 passes of 512 entries) against the oracle: payload and coded bytes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits, k", [(2, k) for k in (4, 8, 12, 16, 20, 36, 60, 68, 124, 132, 256, 260, 508, 512, 516, 1024,
                                                      1028, 2048, 2052, 4092, 4096)]
                         + [(b, k) for b in (1, 3, 4) for k in (8, 16, 24, 64, 72, 248, 504, 520, 1032, 2056, 4096)])
def test_codes_at_mapping_edges(oracle, bits, k):
    from paper_2508_15706_amd import binding as sl
    # chunk counts 67, 1 and 9: no multiple of the chunks that share a wave
    descs, off = [], 0
    for chunks in (67, 1, 9):
        descs.append((1, 4096 * chunks, off, sl.SL_LAYOUT_FLAT))
        off += 4096 * chunks
    rng = np.random.default_rng(1000 * bits + k)
    delta = rng.standard_t(3, off).astype(np.float32)         # far values, so that every bin is met
    plan = sl.sl_plan_create_bits(descs, k, bits)
    pay, ws = sl.alloc_payload(plan), sl.alloc_workspace(plan)
    coded = torch.zeros(sl.sl_rice_max_bytes(plan), dtype=torch.uint8, device="cuda")
    e = torch.zeros(off, dtype=torch.float32, device="cuda")
    sl.sl_compress_coded(plan, e, torch.from_numpy(delta).cuda(), 0.95, pay, coded, ws)
    torch.cuda.synchronize()
    e_ref = np.zeros(off, np.float32)
    want = oracle.compress_b(descs, k, bits, e_ref, delta, 0.95)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)
    size = sl.coded_size(coded)
    assert np.array_equal(coded[:size].cpu().numpy(), oracle.rice_encode_b(descs, k, bits, want))
    assert np.array_equal(e.cpu().numpy().view(np.uint32), e_ref.view(np.uint32))

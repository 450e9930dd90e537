"""The words in front of a coding group, summed over the whole list: as many groups as fill the workgroup and the blocks of the scan
and as the placement still takes in one launch, one less and one more, in tensors that end inside blocks.  Both writers of the coded
format, against the oracle, byte for byte."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (chunks of each tensor)
LISTS = [[1] * n for n in (1, 15, 16, 17, 250, 251, 1023, 1024, 1025, 2047, 2048, 2049, 3073)]
LISTS += [[17] * 60 + [16] * 904 + [1], [16 * 1030 + 5, 3, 40]]


@pytest.mark.parametrize("bits", [2, 32])
@pytest.mark.parametrize("chunks", LISTS, ids=lambda c: f"{len(c)}x{c[0]}")
def test_group_offsets(oracle, chunks, bits):
    from paper_2508_15706_amd import binding as sl
    k = 8
    descs, n = [], 0
    for c in chunks:
        descs.append((1, 4096 * c, n, 0))
        n += 4096 * c
    rng = np.random.default_rng(n)
    delta = rng.standard_normal(n, dtype=np.float32) * np.float32(1e-3)
    delta.reshape(-1, 4096)[::5, :k] *= np.float32(1e3)         # runs of other lengths
    want = oracle.compress_b(descs, k, bits, np.zeros(n, np.float32), delta, 0.95, ef_frozen=True)
    coded = oracle.rice_encode_b(descs, k, bits, want)
    plan = sl.sl_plan_create_bits(descs, k, bits)
    pay, out = sl.alloc_payload(plan), torch.full((sl.sl_rice_max_bytes(plan) + 64,), 0xCD, dtype=torch.uint8, device="cuda")
    ws = sl.alloc_workspace(plan)
    sl.sl_compress_coded(plan, None, torch.from_numpy(delta).cuda(), 0.95, pay, out, ws, flags=sl.SL_COMPRESS_EF_FROZEN)
    assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)
    assert np.array_equal(out[:coded.size].cpu().numpy(), coded)
    out.fill_(0xCD)
    sl.sl_rice_encode(plan, pay, out, ws)
    assert np.array_equal(out[:coded.size].cpu().numpy(), coded)
    assert bool((out[coded.size:] == 0xCD).all())

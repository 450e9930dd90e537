"""sl_rice_encode / sl_rice_decode where the number of chunks per wave and of entries per lane changes: densities on both
sides of every step, tensors that end inside a wave's chunks and inside a coding group, records of odd sizes, and supports
whose gaps are far from even (a lane's codes span more than 64 bits).  Against the oracle, byte for byte."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [(k, 2) for k in (4, 12, 28, 32, 36, 40, 64, 68, 72, 132, 136, 256, 260, 264, 512, 516, 520, 1024, 1416, 1424, 4096)]
CASES += [(8, 1), (24, 1), (520, 1), (8, 3), (40, 3), (136, 3), (16, 4), (128, 4), (264, 4), (8, 32), (72, 32), (1024, 32)]
CASES += [(3968, 32), (3976, 32), (4096, 32)]           # the last densities whose fixed records fit four waves' LDS, and beyond


@pytest.mark.parametrize("k, bits", CASES)
def test_transcode_edges(oracle, k, bits):
    from paper_2508_15706_amd import binding as sl
    descs, off = [], 0
    for chunks in (1, 3, 16, 21, 38):
        descs.append((1, 4096 * chunks, off, 0))
        off += 4096 * chunks
    descs.append((128, 192, off, 1))
    n = off + 128 * 192
    rng = np.random.default_rng(10 * k + bits)
    delta = rng.normal(0, 1e-3, n).astype(np.float32)
    x = delta[:off].reshape(-1, 4096)
    x[1::4, :max(k // 2, 1)] *= 1e3                     # one cluster and the rest of the entries elsewhere
    x[2::4, -k:] *= 1e3                                 # everything at the end: the largest first gap
    x[3::4, :k // 2] *= 1e3                             # both ends
    x[3::4, 4096 - (k - k // 2):] *= 1e3
    want = oracle.compress_b(descs, k, bits, np.zeros(n, np.float32), delta, 0.95, ef_frozen=True)
    coded = oracle.rice_encode_b(descs, k, bits, want)
    plan = sl.sl_plan_create_bits(descs, k, bits)
    cap = sl.sl_rice_max_bytes(plan)
    out = torch.full((cap + 64,), 0xCD, dtype=torch.uint8, device="cuda")
    pay = torch.from_numpy(np.concatenate([want, np.zeros(16, np.uint8)])).cuda()
    sl.sl_rice_encode(plan, pay, out, sl.alloc_workspace(plan))
    assert sl.coded_size(out) == coded.size
    assert np.array_equal(out[:coded.size].cpu().numpy(), coded)
    assert bool((out[coded.size:] == 0xCD).all())
    back = torch.full((plan.payload_bytes + 64,), 0xEE, dtype=torch.uint8, device="cuda")
    sl.sl_rice_decode(plan, out, coded.size, back)
    assert np.array_equal(back[:plan.payload_bytes].cpu().numpy(), want)
    assert bool((back[plan.payload_bytes:] == 0xEE).all())

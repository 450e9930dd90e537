"""Both aggregates at the edges of their decode layouts (lanes per worker, workers side by side in a wave,
steps per worker, batches, records at odd addresses), with and without the global momentum, on spread and on
clustered supports, against the oracle's aggregate of the same payloads."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def supports(rng, n, k, kind):
    """A pseudo-gradient whose Top-k support per run of 4096 is spread, or split between both ends of the
    run (one gap that is longer than any window of quotient bits), or one block."""
    d = rng.normal(0, 1e-3, n).astype(np.float32)
    if kind != "spread":
        big = rng.normal(0, 1, n).astype(np.float32)
        big += np.copysign(np.float32(1.0), big)
        j = np.arange(n) % 4096
        keep = (j < k // 2) | (j >= 4096 - (k - k // 2)) if kind == "ends" else (j >= 777) & (j < 777 + k)
        d = np.where(keep, big, d).astype(np.float32)
    return d


@pytest.mark.parametrize("k, R", [(8, 64), (20, 64), (48, 64), (56, 61), (64, 49), (72, 45), (96, 33), (100, 40), (128, 25),
                                  (136, 17), (144, 3), (168, 13), (176, 12), (192, 64), (248, 9), (256, 1), (256, 18),
                                  (264, 5), (504, 6), (512, 9), (520, 4), (1024, 9), (1032, 5), (1416, 3), (1424, 2),
                                  (2048, 3), (2056, 2), (3072, 2), (4088, 2), (4096, 2)])
def test_aggregates_at_layout_edges(oracle, k, R):
    from paper_2508_15706_amd import binding as sl
    # full runs, tiles and a partial tile that still holds k elements
    descs, off = [], 0
    for r, c, lay in ((1, 3 * 4096, 0), (128, 64, 1), (127, 128, 1) if k <= 4032 else (64, 64, 1)):
        descs.append((r, c, off, lay))
        off += (r * c + 63) // 64 * 64
    rng = np.random.default_rng(17 * k + R)
    plan = sl.sl_plan_create(descs, k)
    theta0 = rng.normal(0, 0.02, off).astype(np.float32)
    refs, plain, wires, sizes = [], [], [], []
    for r in range(R):
        d = supports(rng, off, k, ("spread", "ends", "block")[r % 3])
        refs.append(oracle.compress(descs, k, np.zeros(off, np.float32), d, 0.95))
        plain.append(torch.from_numpy(np.concatenate([refs[-1], np.zeros(16, np.uint8)])).cuda())
        wire = oracle.rice_encode(descs, k, refs[-1])
        wires.append(torch.from_numpy(wire).cuda())
        sizes.append(wire.size)
    want = theta0.copy()
    oracle.decompress_avg_apply(descs, k, want, refs, 0.8)
    for call in ("plain", "coded"):
        theta = torch.from_numpy(theta0.copy()).cuda()
        if call == "plain":
            sl.sl_decompress_avg_apply(plan, theta, plain, 0.8)
        else:
            sl.sl_decompress_avg_apply_coded(plan, theta, wires, sizes, 0.8)
        torch.cuda.synchronize()
        assert np.array_equal(theta.cpu().numpy().view(np.uint32), want.view(np.uint32)), call
    # the same with the global momentum: instantiations of their own, with the momentum's loads beside the decode's
    mom0 = rng.normal(0, 1e-3, off).astype(np.float32)
    want, mom_want = theta0.copy(), mom0.copy()
    oracle.decompress_avg_apply_nesterov_b(descs, k, 2, want, mom_want, refs, 0.8, 0.9)
    for call in ("plain", "coded"):
        theta, mom = torch.from_numpy(theta0.copy()).cuda(), torch.from_numpy(mom0.copy()).cuda()
        if call == "plain":
            sl.sl_decompress_avg_apply_nesterov(plan, theta, mom, plain, 0.8, 0.9)
        else:
            sl.sl_decompress_avg_apply_nesterov_coded(plan, theta, mom, wires, sizes, 0.8, 0.9)
        torch.cuda.synchronize()
        assert np.array_equal(theta.cpu().numpy().view(np.uint32), want.view(np.uint32)), call + ", momentum: theta"
        assert np.array_equal(mom.cpu().numpy().view(np.uint32), mom_want.view(np.uint32)), call + ", momentum"
    back = torch.full((plan.payload_bytes,), 0xEE, dtype=torch.uint8, device="cuda")
    for r in range(min(R, 3)):
        sl.sl_rice_decode(plan, wires[r], sizes[r], back)
        torch.cuda.synchronize()
        assert np.array_equal(back.cpu().numpy(), refs[r]), f"worker {r} decoded"


@pytest.mark.parametrize("bits, k, R", [(b, k, R) for b in (1, 3, 4, 32) for k, R in ((16, 64), (24, 43), (32, 33), (64, 17), (72, 15), (72, 64),
                                                                                      (80, 13), (96, 11), (128, 9), (168, 7), (256, 5))]
                         + [(2, 16, 64), (2, 72, 15), (2, 72, 64), (2, 160, 7)])
def test_coded_aggregate_batches(oracle, bits, k, R):
    """The coded aggregate where the number of workers staged at a time is decided: fewer than a pass of the decode
    holds, just as many, whole passes and a remainder that waits for the next batch; with and without momentum."""
    from paper_2508_15706_amd import binding as sl
    descs, off = [], 0
    for r, c, lay in ((1, 2 * 4096, 0), (64, 64, 1), (127, 64, 1)):
        descs.append((r, c, off, lay))
        off += (r * c + 63) // 64 * 64
    rng = np.random.default_rng(1000 * bits + 17 * k + R)
    plan = sl.sl_plan_create_bits(descs, k, bits)
    theta0, mom0 = rng.normal(0, 0.02, off).astype(np.float32), rng.normal(0, 1e-3, off).astype(np.float32)
    refs, wires, sizes = [], [], []
    for r in range(R):
        d = supports(rng, off, k, ("spread", "ends", "block")[r % 3])
        refs.append(oracle.compress_b(descs, k, bits, np.zeros(off, np.float32), d, 0.95))
        wire = oracle.rice_encode_b(descs, k, bits, refs[-1])
        wires.append(torch.from_numpy(wire).cuda())
        sizes.append(wire.size)
    want = theta0.copy()
    oracle.decompress_avg_apply_b(descs, k, bits, want, refs, 0.8)
    theta = torch.from_numpy(theta0.copy()).cuda()
    sl.sl_decompress_avg_apply_coded(plan, theta, wires, sizes, 0.8)
    torch.cuda.synchronize()
    assert np.array_equal(theta.cpu().numpy().view(np.uint32), want.view(np.uint32))
    want, mom_want = theta0.copy(), mom0.copy()
    oracle.decompress_avg_apply_nesterov_b(descs, k, bits, want, mom_want, refs, 0.8, 0.9)
    theta, mom = torch.from_numpy(theta0.copy()).cuda(), torch.from_numpy(mom0.copy()).cuda()
    sl.sl_decompress_avg_apply_nesterov_coded(plan, theta, mom, wires, sizes, 0.8, 0.9)
    torch.cuda.synchronize()
    assert np.array_equal(theta.cpu().numpy().view(np.uint32), want.view(np.uint32)), "theta with momentum"
    assert np.array_equal(mom.cpu().numpy().view(np.uint32), mom_want.view(np.uint32)), "momentum"

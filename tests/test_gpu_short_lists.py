"""Lists on both sides of the rules for short ones: statistics found by the code kernel itself (tensors of up to 1024 chunks,
lists of up to 8192, at most two tensors in any code wave), and the lengths where workgroups of a wave-per-chunk aggregate change between one chunk and four (680, 1025, 1364;
those aggregates themselves: test_gpu_wave_per_chunk.py).  Payload, coded bytes, e and both
aggregates against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [(64, 2, [1024]), (64, 2, [1025]), (16, 4, [3, 1024, 1, 17]), (8, 1, [1] * 40), (8, 2, [64] * 5), (8, 2, [63] * 5),
         (4, 2, [250, 1]), (520, 3, [65, 2]), (1024, 2, [9, 1, 1]), (32, 2, [255, 256, 257]), (16, 2, [1024] * 8),
         (16, 2, [1024] * 8 + [1]), (16, 2, [4095]), (40, 32, [20])]
# two and three tensors in a code wave; a run of one-chunk tensors beside long ones; fewer chunks than a code wave takes; coded
# placement in launches of its own behind statistics found by the code kernel
CASES += [(8, 2, [32] * 6), (8, 2, [21] * 6), (64, 4, [15, 1, 7, 9]), (8, 2, [1000] * 4 + [1] * 57), (64, 2, [1]), (16, 1, [3, 2]),
          (64, 4, [8] * 170), (264, 4, [2] * 200)]
# where workgroups change between one chunk and four, at a low and a high density
CASES += [(64, 2, [679, 1]), (64, 2, [681]), (128, 2, [1025, 339]), (136, 2, [600, 764]), (64, 2, [1365])]


@pytest.mark.parametrize("k, bits, sizes", CASES, ids=lambda v: str(v).replace(" ", "")[:24])
def test_short_list_edges(oracle, k, bits, sizes):
    from paper_2508_15706_amd import binding as sl
    descs, n = [], 0
    for c in sizes:
        descs.append((64 * c, 64, n, 1) if c % 2 else (1, 4096 * c, n, 0))
        n += 4096 * c
    rng = np.random.default_rng(1000 * k + sum(sizes) + bits)
    e0 = rng.normal(0, 1e-3, n).astype(np.float32)
    delta = rng.normal(2e-4, 1e-3, n).astype(np.float32)
    delta[:4096] = e0[:4096] = 0                        # an all-zero chunk: ties
    plan = sl.sl_plan_create_bits(descs, k, bits)
    ws = sl.alloc_workspace(plan)
    want_e = e0.copy()
    want = oracle.compress_b(descs, k, bits, want_e, delta, 0.95)
    coded = oracle.rice_encode_b(descs, k, bits, want)
    theta0 = rng.normal(0, 0.02, n).astype(np.float32)
    want_theta = theta0.copy()
    oracle.decompress_avg_apply_b(descs, k, bits, want_theta, [want, want], 0.8)
    d = torch.from_numpy(delta).cuda()
    for wire in (False, True):
        e, theta = torch.from_numpy(e0).cuda(), torch.from_numpy(theta0).cuda()
        pay = torch.full((plan.payload_bytes + 64,), 0xAB, dtype=torch.uint8, device="cuda")
        if wire:
            out = torch.full((sl.sl_rice_max_bytes(plan) + 64,), 0xCD, dtype=torch.uint8, device="cuda")
            sl.sl_compress_coded(plan, e, d, 0.95, pay, out, ws)
            assert sl.coded_size(out) == coded.size
            assert np.array_equal(out[:coded.size].cpu().numpy(), coded)
            assert bool((out[coded.size:] == 0xCD).all())
            sl.sl_decompress_avg_apply_coded(plan, theta, [out, out], [coded.size, out.numel()], 0.8)
        else:
            sl.sl_compress(plan, e, d, 0.95, pay, ws)
            sl.sl_decompress_avg_apply(plan, theta, [pay, pay], 0.8)
        assert np.array_equal(pay[:plan.payload_bytes].cpu().numpy(), want)
        assert bool((pay[plan.payload_bytes:] == 0xAB).all())
        assert np.array_equal(e.cpu().numpy().view(np.uint32), want_e.view(np.uint32))
        assert np.array_equal(theta.cpu().numpy().view(np.uint32), want_theta.view(np.uint32))

"""The fused front half of a greedy pass: both weight types, short and long blocks
(needs an MI355X).

An all-greedy call runs selection, Fuse, Mix and the first Trans product as one
kernel; an all-zero temperature vector sends the same rows through the separate
kernels.  Both add in the same order, so every output agrees bit for bit.
Sizes: blocks on both sides of 8 positions and at 1, 2 and 16, and batches on
both sides of the one-round rule (256 CUs: 24 fp32 or 32 bf16 sequences of up to 8
positions, 8 of longer ones)."""
import numpy as np
import pytest

from _parity import check_refine, custom_problem, make_refiner, run_device, upload

pytestmark = pytest.mark.gpu

STRESS = dict(W_e=1.0, W_r=0.3, L=0.3, W_in=0.08, W_1=0.08, W_2=0.06)


@pytest.mark.parametrize("dtype,B,batch,seeded", [
    ("f32", 1, 1, False), ("f32", 2, 3, True), ("f32", 8, 1, True), ("f32", 8, 24, False),
    ("f32", 8, 25, False), ("f32", 9, 2, False), ("f32", 9, 9, True), ("f32", 16, 1, False),
    ("f32", 16, 8, True), ("bf16", 1, 2, False), ("bf16", 7, 4, True), ("bf16", 8, 2, False),
    ("bf16", 8, 32, False), ("bf16", 8, 33, True), ("bf16", 16, 8, False), ("bf16", 16, 9, False)])
def test_fused_pass_equals_separate_kernels(dtype, B, batch, seeded):
    import torch
    print(f"fused pass: {dtype} B={B} batch={batch} seeded={seeded}", flush=True)
    prob = custom_problem(dtype, H=512, V=2000, B=B, batch=batch, K=5, sigmas=STRESS,
                          seed=60 + B, seed_given=seeded)
    ref, dev = make_refiner(prob), upload(prob)
    assert dev["temp"] is None
    sep = dict(dev)
    sep["temp"] = torch.zeros(batch, dtype=torch.uint8, device="cuda")
    sep["u_draft"] = torch.zeros((batch, B), dtype=torch.float32, device="cuda")
    for early in (False, True):
        fused = run_device(ref, prob, dev, early_exit=early)
        split = run_device(ref, prob, sep, early_exit=early)
        assert np.array_equal(fused.ids, split.ids)
        assert np.array_equal(fused.iters, split.iters)
        if not early:
            assert np.array_equal(fused.traj, split.traj)
            tally, _ = check_refine(prob, fused)
            assert tally.exact >= 0.9 * tally.decisions
        assert np.array_equal(fused.logits.view(np.uint32), split.logits.view(np.uint32))

"""The selection of a pass made by the next pass's Fuse + Mix kernel (needs an
MI355X).

Batches that the fused greedy pass does not take select the tokens of passes
0 .. K-2 inside the following pass's first kernel and those of the last pass in
a kernel of their own.  So the iterate that a K-pass call records after pass j
equals the ids of a j-pass call, token for token, and the early exit changes
neither ids nor pass counts.  Sizes: one and several key rows (V = 300 to
20001), blocks of 1, 16, 17 and 32 positions, greedy and sampled sequences side
by side, one sequence and several."""
import numpy as np
import pytest

from _parity import check_refine, custom_problem, make_refiner, run_device, upload

pytestmark = pytest.mark.gpu

STRESS = dict(W_e=1.0, W_r=0.3, L=0.3, W_in=0.08, W_1=0.08, W_2=0.06)


@pytest.mark.parametrize("dtype,V,B,batch,temp,seeded", [
    ("bf16", 300, 1, 3, "sample", False), ("bf16", 2000, 16, 3, "mixed", True),
    ("bf16", 20001, 17, 4, "mixed", False), ("bf16", 20001, 32, 5, "greedy", False),
    ("f32", 300, 32, 2, "mixed", False), ("f32", 2000, 16, 9, "greedy", True),
    ("f32", 6113, 7, 5, "sample", False)])
def test_iterates_equal_shorter_calls(dtype, V, B, batch, temp, seeded):
    print(f"pass select: {dtype} V={V} B={B} batch={batch} {temp}", flush=True)
    K = 5
    prob = custom_problem(dtype, H=512, V=V, B=B, batch=batch, K=K, sigmas=STRESS, temp=temp,
                          seed=70 + B, seed_given=seeded)
    ref, dev = make_refiner(prob), upload(prob)
    whole = run_device(ref, prob, dev)
    for j in range(K):
        part = run_device(ref, prob, dev, K=j)
        assert np.array_equal(whole.traj[j], part.ids)
        assert np.array_equal(whole.traj[:j + 1], part.traj[:j + 1])
    early = run_device(ref, prob, dev, early_exit=True)
    assert np.array_equal(early.ids, whole.ids) and np.array_equal(early.iters, whole.iters)
    assert np.array_equal(early.logits.view(np.uint32), whole.logits.view(np.uint32))
    tally, _ = check_refine(prob, whole)
    assert tally.exact >= 0.9 * tally.decisions

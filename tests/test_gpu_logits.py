"""The refined logits that a refine writes: from the last pass alone, as rows of
any vocabulary size and alignment (needs an MI355X).

The many-position Read writes a row's values straight from its accumulators
where 16-byte stores are possible, and through a store buffer two tiles at a
time elsewhere (a vocabulary that is not a multiple of 4, a misaligned buffer);
both write the same values, so the results are compared bit for bit, and one of
them with the oracle within the device error bound.
"""
import numpy as np
import pytest

from _parity import custom_problem, make_refiner, run_device, upload

STRESS = dict(W_e=1.0, W_r=0.3, L=0.3, W_in=0.08, W_1=0.08, W_2=0.06)


# positions: one stream block, and 1 to 4 position blocks per wave of the
# many-position Read with full and partial last blocks; vocabularies: a
# multiple of 4, odd tails, and fewer tiles than the chip has workgroups
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,V,B,batch", [
    ("bf16", 1000, 16, 1), ("bf16", 4100, 16, 3), ("bf16", 4099, 16, 3), ("bf16", 4097, 13, 20),
    ("bf16", 40004, 16, 17), ("bf16", 40001, 24, 16), ("bf16", 33002, 32, 33),
    ("bf16", 33004, 32, 34), ("f32", 3001, 11, 3), ("f32", 4100, 16, 4)])
def test_logit_rows(dtype, V, B, batch):
    import torch
    from test_gpu_parity import _full_check
    print(f"logit rows: {dtype} V={V} B={B} batch={batch}", flush=True)
    prob = custom_problem(dtype, H=256, V=V, B=B, batch=batch, K=5, sigmas=STRESS,
                          temp="mixed" if batch > 1 else "sample", seed=700 + V % 97 + batch)
    ref, dev = make_refiner(prob), upload(prob)
    if prob.batch <= 4:
        _full_check(prob, ref, dev, min_exact=0.0)
    fixed = run_device(ref, prob, dev)
    # sequences stop at passes of their own; the logits are still everyone's
    early = run_device(ref, prob, dev, early_exit=True)
    assert np.array_equal(early.ids, fixed.ids)
    assert np.array_equal(early.logits.view(np.uint32), fixed.logits.view(np.uint32))
    # a caller's buffer that is not 16-byte aligned, with guard values around it
    from paper_2608_02438_amd.xpress import RefineOut
    n = batch * B * V
    for shift in (1, 2):
        flat = torch.full((n + 8,), 7.5, dtype=torch.float32, device="cuda")
        out = RefineOut(ids=torch.empty((batch, B), dtype=torch.int32, device="cuda"),
                        iters=torch.empty((batch,), dtype=torch.int32, device="cuda"),
                        logits=flat[shift:shift + n].view(batch, B, V), traj=None)
        ref.refine_block(dev["hidden"], dev["anchor"], seed_ids=dev["seed_ids"], temp=dev["temp"],
                         u_draft=dev["u_draft"], K=prob.K, write_logits=True, out=out)
        got = flat.cpu().numpy()
        assert np.array_equal(got[shift:shift + n].view(np.uint32),
                              fixed.logits.reshape(-1).view(np.uint32))
        assert (got[:shift] == 7.5).all() and (got[shift + n:] == 7.5).all()
    # K = 0: the base logits as rows
    base = run_device(ref, prob, dev, K=0)
    h = prob.inp.h.astype(np.float32) if dtype == "f32" else \
        (prob.inp.h.astype(np.uint32) << 16).view(np.float32)
    w = prob.weights["W_lm"] if dtype == "f32" else \
        (prob.weights["W_lm"].astype(np.uint32) << 16).view(np.float32)
    want = h.reshape(-1, prob.H).astype(np.float64) @ w.astype(np.float64).T
    # fp32 sums of H products: 6 u sqrt(H) |w_v| |h_k| (the probabilistic bound of the parity tests)
    bound = 6 * 2.0 ** -24 * np.sqrt(prob.H) * np.linalg.norm(h.reshape(-1, prob.H), axis=1)[:, None] \
        * np.linalg.norm(w, axis=1)[None, :] + 2.0 ** -24 * np.abs(want)
    assert (np.abs(base.logits.reshape(-1, V) - want) <= bound).all()


# truncating rows keep their logits in the workspace for every pass; the others
# (greedy and plain sampled ones in the same batch) are written once
@pytest.mark.gpu
@pytest.mark.parametrize("V,batch,early", [(4100, 5, False), (4099, 5, True), (5001, 1, True)])
def test_logit_rows_with_truncation(V, batch, early):
    print(f"truncated logit rows: V={V} batch={batch} early={early}", flush=True)
    prob = custom_problem("bf16", H=256, V=V, B=9, batch=batch, K=4, sigmas=STRESS, temp="sample",
                          seed=800 + batch, top_k=[7, 0, 0, 3, 0][:batch],
                          top_p=[1.0, 0.7, 1.0, 0.9, 1.0][:batch])
    if batch > 1:
        prob.inp.temp[-1] = 0
    ref, dev = make_refiner(prob), upload(prob)
    from test_gpu_parity import _full_check
    run, _ = _full_check(prob, ref, dev, min_exact=0.0)
    again = run_device(ref, prob, dev, early_exit=early)
    assert np.array_equal(again.ids, run.ids)
    assert np.array_equal(again.logits.view(np.uint32), run.logits.view(np.uint32))

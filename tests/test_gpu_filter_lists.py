"""Truncated sampling where its candidate list begins and ends, against the
fp64 oracle (needs an MI355X): top-k of 1, at and beyond the number of
vocabulary units, at and beyond the list's limit (which fall back to the
general way), ties that overflow the list, and top-p alone and inside top-k, on
the one-block stream, the GEMM and the fp32 kernels."""
import numpy as np
import pytest

from _parity import custom_problem, make_refiner, run_device, upload
from test_gpu_filter import _check, _verify

pytestmark = pytest.mark.gpu

STRESS = dict(W_e=1.0, W_r=0.3, L=0.3, W_in=0.08, W_1=0.08, W_2=0.06)


# V = 20011: 1251 tiles, 2048 Read units of at most one tile (797 of them empty),
# 314 LM-head GEMM units (or 256 of the stream) and 313 target units, so k = 256,
# 313 and 314 end the list in one kernel and not in another; 1024 is the list's
# largest k, in the Read's rows too
@pytest.mark.parametrize("dtype,B,batch", [("bf16", 5, 2), ("bf16", 6, 8), ("f32", 5, 4)])
@pytest.mark.parametrize("ks", [[1, 2, 255, 256], [257, 313, 314, 315],
                                [1023, 1024, 1025, 1256], [1257, 20010, 0, 64]])
def test_top_k_limits(dtype, B, batch, ks):
    ks = (ks * batch)[:batch]
    ps = [1.0, 0.9, 0.6, 1.0, 0.3, 0.99, 1.0, 0.8][:batch]
    print(f"top-k limits {dtype} B={B} batch={batch} k={ks} p={ps}", flush=True)
    prob = custom_problem(dtype, H=256, V=20011, B=B, batch=batch, K=3, sigmas=STRESS,
                          temp="sample", seed=60 + ks[0] + batch,
                          tau=np.linspace(0.6, 1.4, batch), top_k=ks, top_p=ps)
    ref, dev = make_refiner(prob), upload(prob)
    run = _check(prob, ref, dev, max_excused=2)
    again = run_device(ref, prob, dev, early_exit=True)
    assert np.array_equal(again.ids, run.ids)


# V = 6397: 400 tiles, 800 Read units of which half are empty, 100 LM-head GEMM units
# (or 256 of the stream) and 100 target units: the Read's list ends at its own number
# of units, and past the 400 that hold tokens its bound is the empty ones' maximum
@pytest.mark.parametrize("dtype,B,batch", [("bf16", 5, 2), ("bf16", 6, 8), ("f32", 5, 4)])
@pytest.mark.parametrize("ks", [[99, 100, 101, 256], [399, 400, 401, 512],
                                [799, 800, 801, 1024]])
def test_top_k_at_the_read_units(dtype, B, batch, ks):
    ks = (ks * batch)[:batch]
    ps = [0.9, 1.0, 0.7, 1.0, 1.0, 0.95, 0.5, 1.0][:batch]
    print(f"top-k at the read units {dtype} B={B} batch={batch} k={ks} p={ps}", flush=True)
    prob = custom_problem(dtype, H=256, V=6397, B=B, batch=batch, K=3, sigmas=STRESS,
                          temp="sample", seed=160 + ks[0] + batch,
                          tau=np.linspace(0.6, 1.4, batch), top_k=ks, top_p=ps)
    _check(prob, make_refiner(prob), upload(prob), max_excused=2)


# every logit equal: k tokens tie with all others, the list overflows, and the
# top-p cut falls inside the tie
@pytest.mark.parametrize("V,k,p", [(5003, 3, 1.0), (5003, 3, 0.25), (300, 7, 0.5), (17, 2, 0.5)])
def test_ties_overflow(V, k, p):
    print(f"ties V={V} k={k} p={p}", flush=True)
    prob = custom_problem("bf16", H=256, V=V, B=4, batch=5, K=2,
                          sigmas=dict(W_lm=0.0, W_r=0.0), temp="sample", seed=90 + V % 50,
                          top_k=k, top_p=p)
    ref, dev = make_refiner(prob), upload(prob)
    _check(prob, ref, dev, max_excused=0)


# a NaN beside the row's largest logit, a row of NaN (of the sign that sorts below
# every number), more NaN than top-k keeps on the general way: no token has mass and
# the choice is the first of the vocabulary, as the general way makes it; the last
# sequence has none of them and keeps its token
def test_target_rows_with_nan():
    import torch
    print("target rows with NaN, V=5004 k=[1, 4, 2000, 50]", flush=True)
    prob = custom_problem("bf16", H=256, V=5004, B=4, batch=4, K=2, sigmas=STRESS,
                          temp="sample", seed=95, top_k=[1, 4, 2000, 50], top_p=1.0)
    ref, dev = make_refiner(prob), upload(prob)
    run = run_device(ref, prob, dev)
    target_ids = prob.inp.target_ids(run.ids)
    n0, nx0 = _verify(ref, prob, run, dev, target_ids)
    tl = prob.inp.target_logits.copy()
    for k in range(prob.B + 1):
        tl[0, k, tl[0, k].argmax() ^ 1] = np.nan
    tl[1] = np.array([0xFFC00000], dtype=np.uint32).view(np.float32)[0]
    tl[2, :, :2500] = np.nan
    dev["target_logits"] = torch.from_numpy(tl).cuda()
    n, nx = _verify(ref, prob, run, dev, target_ids)
    print(f"  n={n.tolist()} next={nx.tolist()}", flush=True)
    assert n[:3].tolist() == [0, 0, 0] and nx[:3].tolist() == [0, 0, 0]
    assert (n[3], nx[3]) == (n0[3], nx0[3])

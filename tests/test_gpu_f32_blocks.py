"""The fp32 refiner over several position blocks at once (needs an MI355X).

A call of more than 16 positions multiplies up to four 16-position blocks with
every tile of W_lm and of W_r; each product keeps the order of additions of the
one-block kernels, so a batch equals its sequences run one by one, bit for bit.
Sizes: two to four blocks in one or two workgroup columns with partial last
blocks, units of two tiles up to several groups of tiles, a vocabulary one row
over a tile, k slices of 1, 2 and 16 load units, and the vocabularies on both
sides of the rule that sends a call there."""
import numpy as np
import pytest

from _parity import custom_problem, make_refiner, run_device, upload

pytestmark = pytest.mark.gpu

STRESS = dict(W_e=1.0, W_r=0.3, L=0.3, W_in=0.08, W_1=0.08, W_2=0.06)


@pytest.mark.parametrize("H,V,B,batch", [
    (256, 6113, 11, 2), (256, 6145, 11, 3), (512, 12289, 16, 4), (512, 40001, 13, 5),
    (256, 70000, 16, 2), (4096, 6200, 9, 2), (256, 6400, 16, 9), (256, 300, 16, 3),
    # the Read's forms: one tile for a wave's one or two units (an odd number of
    # read workgroups, the last vocabularies of both forms and one row more), one to
    # three blocks of it a workgroup, and longer units
    (256, 4000, 16, 5), (256, 4000, 16, 32), (256, 16384, 16, 3), (256, 16384, 16, 12),
    (256, 16385, 16, 3), (256, 32768, 16, 2), (256, 32769, 11, 3), (256, 50000, 16, 5)])
def test_blocks_equal_single_sequences(H, V, B, batch):
    import torch
    print(f"fp32 blocks: H={H} V={V} B={B} batch={batch}", flush=True)
    prob = custom_problem("f32", H=H, V=V, B=B, batch=batch, K=3, sigmas=STRESS, temp="mixed",
                          seed=40 + V % 89 + batch)
    ref, dev = make_refiner(prob), upload(prob)
    for K in (0, 3):
        whole = run_device(ref, prob, dev, K=K)
        for b in range(batch):
            one = ref.refine_block(dev["hidden"][b:b + 1].contiguous(), dev["anchor"][b:b + 1],
                                   temp=dev["temp"][b:b + 1].contiguous(),
                                   u_draft=dev["u_draft"][b:b + 1].contiguous(), K=K,
                                   write_logits=True)
            torch.cuda.synchronize()
            assert np.array_equal(one.ids.cpu().numpy()[0], whole.ids[b])
            assert np.array_equal(one.logits.cpu().numpy()[0].view(np.uint32),
                                  whole.logits[b].view(np.uint32))
    from test_gpu_parity import _full_check
    if H * V <= 4 << 20:
        _full_check(prob, ref, dev, min_exact=0.9)

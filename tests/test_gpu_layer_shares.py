"""The attention's shares of the context against the fp64 oracle (needs an
MI355X): calls whose work list is shorter than the workgroups, one sequence cut
into many parts, many short sequences in one share, shares that end inside the
block's own keys, every group size and both block widths, a sequence beside others
of changing length, and the static-scratch forward where its partials do not fit."""
import numpy as np
import pytest

import oracle as O
import synth
from paper_2608_02438_amd.xpress import LAYER_WEIGHT_NAMES

pytestmark = pytest.mark.gpu


# (KV heads, group, B, contexts): sub-chunks of 64 keys counted per KV head
CASES = [
    (1, 1, 1, [0]),                                   # one sub-chunk in all
    (2, 4, 16, [63, 64, 65, 127]),                    # ends around a sub-chunk's
    (1, 2, 32, [40000]),                              # one segment over every share
    (2, 8, 7, [9000, 0, 1, 5000]),                    # long and empty ones side by side
    (4, 4, 32, [0, 1, 31, 32, 33, 100] * 12),         # several segments in a share
    (8, 1, 16, [300] * 65),                           # more sequences than a wave's lanes
    (2, 8, 32, [2000, 17, 4097]),                     # sixteen waves
]


@pytest.mark.parametrize("nkv,grp,B,ctx", CASES)
@pytest.mark.parametrize("causal", [True, False])
def test_attention_shares(nkv, grp, B, ctx, causal):
    import torch
    from paper_2608_02438_amd.xpress import Layer, device_tensor
    print(f"shares: nkv={nkv} grp={grp} B={B} sequences={len(ctx)} max ctx={max(ctx)} "
          f"causal={causal}", flush=True)
    nh = nkv * grp
    if nh * 128 % 256:                                # n_heads * 128: a multiple of 256
        nkv, nh = 2 * nkv, 2 * nh
    batch, cmax = len(ctx), max(max(ctx), 1)
    w = synth.scaled(synth.configs.QWEN_B1, index=970 + nkv + grp, H=256, B=B, batch=batch,
                     n_heads=nh, n_kv_heads=nkv, ffn=256, ctx_len=None, ctx_len_range=None)
    weights = synth.make_layer_weights(w)
    inp = synth.make_layer_inputs(w, c_max=cmax)
    inp.ctx_len = np.array(ctx, dtype=np.int32)
    dw = {k: device_tensor(weights[k]) for k in LAYER_WEIGHT_NAMES}
    layer = Layer(dw, w.H, nh, nkv, w.ffn, max_batch=batch, max_B=B, max_ctx=cmax)
    args = [device_tensor(a) for a in (inp.x, inp.k_cache, inp.v_cache, inp.ctx_len)]
    h, _ = layer.forward(*args, causal=causal)
    again, _ = layer.forward(*args, causal=causal)
    h, again = h.cpu().numpy(), again.cpu().numpy()
    layer.close()
    assert np.array_equal(h.view(np.uint32), again.view(np.uint32))
    some = sorted({0, 1, 2, 3, batch - 1} & set(range(batch)))
    LP = O.layer_ref.LayerParams.from_arrays(weights, nh, nkv, 128)
    ref = O.layer_ref.layer_forward(LP, inp.x[some], inp.k_cache[some], inp.v_cache[some],
                                    inp.ctx_len[some], causal=causal)
    # the layer parity tests' bar: one bf16 unit at the output's scale
    assert np.abs(h[some] - ref).max() <= max(2e-2, 2.0 ** -8 * np.abs(ref).max())


def test_other_sequences_contexts_move_only_the_summation_order():
    """The shares are cut from all contexts of a call: with the others' lengths a
    sequence is split elsewhere.  Both results lie within the parity bar of the
    oracle; the others' contents change nothing."""
    import torch
    from paper_2608_02438_amd.xpress import Layer, device_tensor
    nkv, nh, B, cmax = 2, 8, 16, 5000
    w = synth.scaled(synth.configs.QWEN_B1, index=983, H=256, B=B, batch=3, n_heads=nh,
                     n_kv_heads=nkv, ffn=256, ctx_len=None, ctx_len_range=None)
    weights = synth.make_layer_weights(w)
    inp = synth.make_layer_inputs(w, c_max=cmax)
    dw = {k: device_tensor(weights[k]) for k in LAYER_WEIGHT_NAMES}
    layer = Layer(dw, w.H, nh, nkv, w.ffn, max_batch=3, max_B=B, max_ctx=cmax)
    x, kc, vc = (device_tensor(a) for a in (inp.x, inp.k_cache, inp.v_cache))
    LP = O.layer_ref.LayerParams.from_arrays(weights, nh, nkv, 128)
    ctx = [4000, 3000, 20]
    ref = O.layer_ref.layer_forward(LP, inp.x[:1], inp.k_cache[:1], inp.v_cache[:1],
                                    np.array(ctx[:1], dtype=np.int32))
    bar = max(2e-2, 2.0 ** -8 * np.abs(ref).max())
    out = []
    for others in ([3000, 20], [0, 5000], [4999, 4999]):
        print(f"shares: contexts {ctx[:1] + others}", flush=True)
        cl = torch.tensor(ctx[:1] + others, dtype=torch.int32, device="cuda")
        h, hb = layer.forward(x, kc, vc, cl)
        out.append(h[0].cpu().numpy())
        assert np.abs(out[-1] - ref[0]).max() <= bar
    print(f"  max difference {max(np.abs(o - out[0]).max() for o in out):.3g}, bar {bar:.3g}",
          flush=True)
    assert all(np.abs(o - out[0]).max() <= bar for o in out)
    # the others' inputs, not their lengths: the same bits
    x2, kc2 = x.clone(), kc.clone()
    x2[1:] *= -1
    kc2[1:] *= -1
    h, _ = layer.forward(x2, kc2, vc, cl)
    assert np.array_equal(h[0].cpu().numpy().view(np.uint32), out[-1].view(np.uint32))
    layer.close()


# more partials than the static scratch holds beside the buffers: fewer shares, one
# part per KV head of a sequence, two parts
@pytest.mark.parametrize("batch,c_max,ns", [(17, 400, 0), (22, 400, 1), (16, 2200, 2)])
def test_static_scratch_without_room_for_the_default(batch, c_max, ns):
    import torch
    from _layer_plan import plans
    from paper_2608_02438_amd.xpress import device_tensor, layer_forward_noalloc, \
        layer_weights_struct
    H, nh, nkv, ffn, B = 256, 64, 8, 256, 17
    plan = plans([(H, nh, nkv, ffn, batch, B, c_max)])[0]
    assert plan.parts > plan.room >= plan.fit_parts and plan.fit_ns == ns
    print(f"static scratch, {batch} x {B} positions, {nh}/{nkv} heads: {plan}", flush=True)
    w = synth.scaled(synth.configs.QWEN_B1, index=990 + ns, H=H, B=B, batch=batch, n_heads=nh,
                     n_kv_heads=nkv, ffn=ffn, ctx_len=None, ctx_len_range=None)
    weights = synth.make_layer_weights(w)
    inp = synth.make_layer_inputs(w, c_max=c_max)
    inp.ctx_len = np.array([[c_max, 0, 64, c_max - 1, 1, 300, 128, 47][b % 8]
                            for b in range(batch)], dtype=np.int32)
    dw = {k: device_tensor(weights[k]) for k in LAYER_WEIGHT_NAMES}
    st = layer_weights_struct(dw, H, nh, nkv, ffn)
    args = [device_tensor(a) for a in (inp.x, inp.k_cache, inp.v_cache, inp.ctx_len)]
    h32 = torch.full((batch, B, H), float("nan"), dtype=torch.float32, device="cuda")
    hb = torch.empty((batch, B, H), dtype=torch.bfloat16, device="cuda")
    layer_forward_noalloc(st, *args, h32, hb)
    got = h32.cpu().numpy()
    layer_forward_noalloc(st, *args, h32, hb)
    assert np.array_equal(got.view(np.uint32), h32.cpu().numpy().view(np.uint32))
    some = [0, 1, 2, 3, 4, batch - 1]
    LP = O.layer_ref.LayerParams.from_arrays(weights, nh, nkv, 128)
    ref = O.layer_ref.layer_forward(LP, inp.x[some], inp.k_cache[some], inp.v_cache[some],
                                    inp.ctx_len[some])
    assert np.isfinite(got).all()
    assert np.abs(got[some] - ref).max() <= max(2e-2, 2.0 ** -8 * np.abs(ref).max())

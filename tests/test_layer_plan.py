"""How a layer forward is cut up, on the CPU: the attention's workgroups with and
without room for their partials, the work list that the attention and its combine
walk, and the parts of k of the projections."""
import random
import shutil

import pytest

from _layer_plan import gemm_plans, plans, walks

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ compiles the rules")

QWEN = (4096, 32, 8, 12288)


def _busy(W, slots):
    return W // -(-W // slots)


def _shapes(n, seed):
    rng = random.Random(seed)
    out = []
    while len(out) < n:
        nkv, grp = rng.choice([1, 2, 4, 8, 16, 32, 64]), rng.choice([1, 2, 4, 8])
        if nkv * grp % 2:
            continue
        B = rng.randint(1, 32)
        out.append((256 * rng.randint(1, 16), nkv * grp, nkv, 256 * rng.randint(1, 48),
                    rng.randint(1, max(1, 700 // B)), B, rng.choice([1, 100, 700, 2000, 2048,
                                                                     2100, 8192, 100000])))
    return out


@pytest.mark.parametrize("batch,B,C_max,least", [
    (27, 16, 2000, 216), (28, 16, 2000, 224), (13, 32, 2000, 104), (14, 32, 2000, 112),
    (28, 16, 8000, 224), (14, 32, 8000, 112)])
def test_static_scratch_never_below_a_workgroup_per_segment(batch, B, C_max, least):
    """Qwen3-8B shape, where the default partials do not fit beside the other
    buffers: one workgroup per KV head of a sequence needs no more of them."""
    p = plans([QWEN + (batch, B, C_max)])[0]
    assert p.parts > p.room and p.fit_parts <= p.room
    assert p.fit_W >= least


def test_plans_over_drawn_shapes():
    cases = _shapes(4000, 1)
    tight = 0
    for c, p in zip(cases, plans(cases)):
        H, nh, nkv, ffn, batch, B, C_max = c
        npb, segs, nsub = -(-B // 16), batch * nkv, -(-(C_max + B) // 64)
        per = npb * (nh // nkv)
        assert p.parts <= p.workspace, c
        assert p.parts == (p.W if p.ns else p.W + segs - 1) * per, c
        assert 1 <= p.W and p.ns <= nsub, c
        if p.room == 0 or segs * per > p.room:           # refused: no room for a part each
            assert p.room == 0 or p.fit_W == 0, c
            continue
        assert p.fit_parts == (p.fit_W if p.fit_ns else p.fit_W + segs - 1) * per, c
        assert p.fit_parts <= p.room, c
        if p.parts <= p.room:
            assert (p.fit_W, p.fit_ns) == (p.W, p.ns), c
        else:
            tight += 1
            assert _busy(p.fit_W, p.slots) >= min(_busy(segs, p.slots), _busy(p.W, p.slots)), c
    assert tight > 50


def test_parts_cover_the_contexts():
    """Every sub-chunk in one part, partial numbers of their own within the plan's
    bound and where the combine looks: default plans and forced ones, contexts
    shorter than C_max, empty ones, more shares than sub-chunks."""
    rng = random.Random(2)
    cases, shapes = [], _shapes(300, 3)
    for s, p in zip(shapes, plans(shapes)):
        nkv, batch, B, C_max = s[2], s[4], s[5], s[6]
        kind = rng.choice(["full", "ragged", "short", "empty"])
        ctx = [{"full": C_max, "ragged": rng.randint(0, C_max), "short": rng.randint(0, 70),
                "empty": 0}[kind] for _ in range(batch)]
        for W, ns in {(p.W, p.ns), (p.fit_W, p.fit_ns), (1, 0), (7, 0), (512, 0),
                      (batch * nkv, 1), (3 * batch * nkv, 3)}:
            if W:
                cases.append((nkv, B, W, ns, [min(c, C_max) for c in ctx]))
    assert all(walks(cases))


def test_parts_of_the_largest_work_list():
    """Beyond 2^22 sub-chunks the shares divide in 64 bits."""
    assert all(walks([(64, 32, 512, 0, [1 << 20] * 5), (64, 32, 511, 0, [0, 1 << 20, 65] * 3),
                      (2, 1, 32, 16, [1 << 20])]))


@pytest.mark.parametrize("K", [4352, 6912, 11008, 12288])
@pytest.mark.parametrize("M", [80, 128])
def test_eight_parts_of_k_for_every_width(K, M):
    """32 tiles of 128 rows on 256 workgroups: eight parts of k, also where K is an
    odd multiple of 256 and the stages of 64 do not divide by eight."""
    bn, S, nk, first = gemm_plans([(4096, 0, 4096, K, M, 1 << 24)])[0]
    assert (bn, S, nk) == (128, 8, K // 64)
    assert max(b - a for a, b in zip(first, first[1:])) == -(-nk // 8)


def test_parts_of_k_cover_it():
    rng = random.Random(4)
    cases = [(N, 0, N, 256 * rng.randint(1, 120), rng.randint(65, 700),
              rng.choice([0, 1 << 20, 1 << 24]))
             for N in (256 * rng.randint(1, 48) for _ in range(3000))]
    uneven = 0
    for c, (bn, S, nk, first) in zip(cases, gemm_plans(cases)):
        K = c[3]
        assert bn in (128, 256) and nk * (64 if bn == 128 else 32) == K, c
        assert first[0] == 0 and first[-1] == nk and len(first) == S + 1, c
        sizes = {b - a for a, b in zip(first, first[1:])}
        assert S == 1 or min(sizes) * K >= 512 * nk, c
        if len(sizes) > 1:                 # a workgroup's tiles lie 8 apart: one part
            uneven += 1
            assert 8 % S == 0 and max(sizes) == min(sizes) + 1, c
    assert uneven > 50

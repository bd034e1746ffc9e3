"""Decode launches of several rounds of workgroups with the rows split evenly over the workgroups (plain mode,
lengths known to the host): against the oracle on ragged batches, and against the fixed-piece launch of the same call.
The small shapes here would normally merge inside one launch; POD_DECODE_FUSED=0 (read when the cache is created)
sends them down the path that large batches take."""
import numpy as np
import pytest
import torch

import paper_2412_02252_amd as pod
from podcase import Case, assert_close

pytestmark = pytest.mark.gpu


def fill_all(c, lens):
    for layer in range(c.L):
        for b, n in enumerate(lens):
            if n:
                c.fill(layer, b, n)


@pytest.mark.parametrize("seed", range(12))
def test_random_ragged_batches_decode_and_steps(seed, monkeypatch):
    """Seeded shapes: head counts, head dim, sink 0, windows, 1..24 sequences of 0..3000 tokens (empty ones, ones
    still inside S + W, long ones): three decode steps, pod_decode_attention, three score-reuse steps, every layer of
    the block."""
    monkeypatch.setenv("POD_DECODE_FUSED", "0")
    rng = np.random.default_rng(9000 + seed)
    d = int(rng.choice([64, 128]))
    Hkv = int(rng.choice([1, 2, 3, 8]))
    rep = int(rng.choice([1, 2, 4, 7] if d == 64 else [1, 2, 4, 8]))
    S = int(rng.choice([0, 4, 16, 64]))
    W = int(rng.choice([8, 40, 128, 500]))
    B = int(rng.integers(1, 25))
    G = int(rng.choice([1, 2, 3]))
    lens = [int(x) for x in rng.choice([0, 1, S + W, S + W + 1, 129, 700, 1500, 3000], size=B)]
    lens = [max(0, n - int(rng.integers(0, 3))) for n in lens]
    c = Case(G, G, Hkv * rep, Hkv, d, S, W, B, 3110, seed=9100 + seed)
    fill_all(c, lens)
    for layer in range(G):      # (the oracle has no notion of an empty entry: here only that such rows come out zero)
        out = c.decode(layer, lens)
        for b, n in enumerate(lens):
            if n == 0:
                assert float(out[b].float().abs().max()) == 0.0
    for s in range(3):
        pos = [n + s for n in lens]
        for layer in range(G):
            assert_close(c.step(layer, pos), c.decode_ref(layer, [p + 1 for p in pos]), f"step {s} layer {layer} lens {lens}")
    ctx = [n + 3 for n in lens]
    for layer in range(G):
        assert_close(c.decode(layer, ctx), c.decode_ref(layer, ctx), f"decode layer {layer} ctx {ctx}")
    # ... and three steps with score reuse: the lowest layer writes its distant logits, the upper layers walk units of
    # twice as many distant rows and read them
    scores = c.gpu.new_score_buffer()
    for s in range(3, 6):
        pos = [n + s for n in lens]
        for layer in range(G):
            assert_close(c.step_reuse(layer, pos, scores), c.decode_ref(layer, [p + 1 for p in pos]), f"reuse step {s} layer {layer} lens {lens}")
    for layer in range(G):
        for b in range(B):
            c.assert_cache_equal(layer, b)
    c.gpu.pod_cache_check()


def test_even_split_and_fixed_pieces_agree(monkeypatch):
    """The same calls through both launch shapes: equal up to the order of the merge."""
    lens = [2900, 17, 0, 1300, 1301, 140, 2048, 5]
    outs = {}
    for even in ("1", "0"):
        monkeypatch.setenv("POD_DECODE_FUSED", "0")
        monkeypatch.setenv("POD_DECODE_EVEN", even)
        c = Case(2, 2, 16, 4, 128, 16, 96, len(lens), 3000, seed=9200, with_oracle_cache=False)
        fill_all(c, lens)
        o = [c.decode(layer, lens).float() for layer in range(2)]
        pos = list(lens)
        o += [c.step(layer, pos).float() for layer in range(2)]
        scores = c.gpu.new_score_buffer()
        pos = [n + 1 for n in lens]
        o += [c.step_reuse(layer, pos, scores).float() for layer in range(2)]
        outs[even] = o
        c.gpu.pod_cache_check()
    for a, b in zip(outs["1"], outs["0"]):
        assert (a - b).abs().max() <= 2.0 ** -7 * b.abs().max()


def test_reuse_steps_follow_plain_steps_and_separate_calls_read_their_logits(monkeypatch):
    """Logits written by an even-split reuse step of the lowest layer are read by the upper layer's reuse step and,
    after the next token's lowest-layer call through the separate entry point, by pod_decode_attention_reuse."""
    monkeypatch.setenv("POD_DECODE_FUSED", "0")
    lens = [1900, 300, 41, 2600]
    c = Case(3, 3, 8, 2, 128, 8, 32, len(lens), 2700, seed=9500)
    fill_all(c, lens)
    scores = c.gpu.new_score_buffer()
    for s in range(4):
        pos = [n + s for n in lens]
        for layer in range(3):
            assert_close(c.step_reuse(layer, pos, scores), c.decode_ref(layer, [p + 1 for p in pos]), f"step {s} layer {layer}")
    pos = [n + 4 for n in lens]
    ctx = [p + 1 for p in pos]
    for layer in range(3):
        c.append(layer, pos)
    for layer in range(3):
        assert_close(c.decode_reuse(layer, ctx, scores), c.decode_ref(layer, ctx), f"separate calls layer {layer}")
    for layer in range(3):
        for b in range(len(lens)):
            c.assert_cache_equal(layer, b)
    c.gpu.pod_cache_check()


@pytest.mark.parametrize("d,Hkv,rep", [(128, 1, 16), (64, 2, 16), (128, 3, 5), (64, 1, 1)])
def test_sixteen_query_heads_per_kv_head_and_other_group_sizes(d, Hkv, rep, monkeypatch):
    """All 16 MFMA columns hold real heads; odd group sizes; a single head."""
    monkeypatch.setenv("POD_DECODE_FUSED", "0")
    lens = [1500, 0, 333, 64, 2047]
    c = Case(2, 2, Hkv * rep, Hkv, d, 4, 60, len(lens), 2100, seed=9600 + rep)
    fill_all(c, lens)
    scores = c.gpu.new_score_buffer()
    for s in range(2):
        pos = [n + s for n in lens]
        for layer in range(2):
            assert_close(c.step(layer, pos), c.decode_ref(layer, [p + 1 for p in pos]), f"step {s} layer {layer}")
    for s in range(2, 4):
        pos = [n + s for n in lens]
        for layer in range(2):
            assert_close(c.step_reuse(layer, pos, scores), c.decode_ref(layer, [p + 1 for p in pos]), f"reuse step {s} layer {layer}")
    ctx = [n + 4 for n in lens]
    for layer in range(2):
        assert_close(c.decode(layer, ctx), c.decode_ref(layer, ctx), f"decode layer {layer}")
    c.gpu.pod_cache_check()


def test_one_long_sequence_among_many_short_ones(monkeypatch):
    """The long sequence is cut into many more parts than any other: its partial count per pair is the launch's."""
    monkeypatch.setenv("POD_DECODE_FUSED", "0")
    lens = [40] * 15 + [6000] + [3] * 8
    c = Case(2, 2, 8, 2, 128, 8, 64, len(lens), 6100, seed=9300)
    fill_all(c, lens)
    for layer in range(2):
        assert_close(c.decode(layer, lens), c.decode_ref(layer, lens), f"layer {layer}")
    pos = list(lens)
    for layer in range(2):
        assert_close(c.step(layer, pos), c.decode_ref(layer, [p + 1 for p in pos]), f"step layer {layer}")
    c.gpu.pod_cache_check()


@pytest.mark.parametrize("d,Hq,Hkv,B,lo,step", [(64, 8, 8, 24, 300, 37), (128, 8, 4, 30, 130, 91), (64, 16, 8, 70, 5, 13), (128, 4, 4, 40, 1, 60)])
def test_parts_of_whole_pairs_and_parts_that_cross(d, Hq, Hkv, B, lo, step, monkeypatch):
    """More units than workgroups: parts padded to whole pairs where they fit, parts that cross from pair to pair where the
    pairs outnumber the workgroups (70 x 8); sequences of a few tokens among them."""
    monkeypatch.setenv("POD_DECODE_FUSED", "0")
    lens = [lo + (step * i * i) % 900 for i in range(B)]
    c = Case(2, 2, Hq, Hkv, d, 8, 64, B, 1210, seed=9350 + B)
    fill_all(c, lens)
    for s in range(2):
        pos = [n + s for n in lens]
        for layer in range(2):
            assert_close(c.step(layer, pos), c.decode_ref(layer, [p + 1 for p in pos]), f"step {s} layer {layer}")
    ctx = [n + 2 for n in lens]
    for layer in range(2):
        assert_close(c.decode(layer, ctx), c.decode_ref(layer, ctx), f"decode layer {layer}")
    c.gpu.pod_cache_check()


@pytest.mark.parametrize("d,Hq,Hkv,B,lo,step", [(64, 8, 8, 24, 300, 37), (64, 16, 4, 44, 130, 91), (64, 6, 2, 80, 3, 77),
                                                (128, 8, 8, 24, 300, 37), (128, 16, 4, 44, 130, 91), (128, 6, 2, 80, 3, 77),
                                                (64, 32, 4, 44, 130, 91), (128, 30, 5, 30, 130, 91), (128, 32, 4, 44, 130, 91),
                                                (64, 64, 4, 44, 130, 91), (128, 64, 4, 44, 130, 91)])
def test_parts_of_whole_pairs_merged_inside(d, Hq, Hkv, B, lo, step):
    """Few query heads' partials per pair: the last part of a pair merges.  Steps, then the same attention again;
    wrong lengths and positions, whose rows come out zero; a graph replayed three times."""
    lens = [lo + (step * i * i) % 900 for i in range(B)]
    c = Case(2, 2, Hq, Hkv, d, 8, 64, B, 1210, seed=9360 + B)
    for call in (pod.CALL_STEP, pod.CALL_ATTENTION):
        pl = c.launched(lens, call)
        assert pl["even"] and pl["merge_inside"], pl
    fill_all(c, lens)
    for s in range(2):
        pos = [n + s for n in lens]
        for layer in range(2):
            assert_close(c.step(layer, pos), c.decode_ref(layer, [p + 1 for p in pos]), f"step {s} layer {layer}")
    ctx = [n + 2 for n in lens]
    refs = [c.decode_ref(layer, ctx) for layer in range(2)]
    for _ in range(2):
        for layer in range(2):
            assert_close(c.decode(layer, ctx), refs[layer], f"decode layer {layer}")
    c.gpu.pod_cache_check()
    qs = [c.decode_queries(layer, ctx, c.dev) for layer in range(2)]
    ctx_dev = torch.tensor(ctx, dtype=torch.int32, device=c.dev)
    out = torch.empty((2,) + tuple(qs[0].shape), dtype=torch.bfloat16, device=c.dev)
    for layer in range(2):
        c.gpu.pod_decode_attention(layer, qs[layer], qs[0] if layer else None, ctx_dev, c.scale, out=out[layer])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for layer in range(2):
            c.gpu.pod_decode_attention(layer, qs[layer], qs[0] if layer else None, ctx_dev, c.scale, out=out[layer])
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        for layer in range(2):
            assert_close(out[layer], refs[layer], f"replay layer {layer}")
    wrong = ctx_dev.clone()
    wrong[1] -= 1
    got = c.gpu.pod_decode_attention(0, qs[0], None, wrong, c.scale)
    with pytest.raises(pod.PodError) as e:
        c.gpu.pod_cache_check()
    assert e.value.code == pod.binding.ERR_STATE
    assert float(got[1].float().abs().max()) == 0.0
    keep = [i for i in range(B) if i != 1]
    assert_close(got[keep], refs[0][keep], "the other sequences")
    k, v = torch.randn((2, B, Hkv, d), device=c.dev).to(torch.bfloat16)
    bad = ctx_dev.clone()
    bad[2] += 1                                                              # sequence 2 holds one token less
    got = c.gpu.pod_decode_step(0, k, v, qs[0], None, bad, c.scale)
    with pytest.raises(pod.PodError) as e:
        c.gpu.pod_cache_check()
    assert e.value.code == pod.binding.ERR_STATE
    assert float(got[2].float().abs().max()) == 0.0 and float(got[3].float().abs().max()) > 0.0


@pytest.mark.parametrize("Hq,Hkv,d,B", [(16, 4, 64, 44), (8, 8, 64, 24), (8, 4, 128, 44)])
def test_empty_sequences_in_the_padded_split(Hq, Hkv, d, B):
    """First, in the middle and last in the batch: no part walks them.  Attention leaves the merge to the second launch, which writes their
    zero rows; a step gives each its first token, which the merging kernel's own workgroup for the pair takes alone; then both
    again with nothing empty."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    lens = [0 if b in (0, 7, 8, B - 1) else 130 + (91 * b * b) % 900 for b in range(B)]
    empty, held = [b for b in range(B) if not lens[b]], [b for b in range(B) if lens[b]]
    assert cus != 256 or (pod.pod_decode_even_launch(cus, Hkv, 72, lens)["padded"] and not pod.pod_decode_plan(cus, B, Hkv, 72, max(lens))["merge_inside"])
    c = Case(2, 2, Hq, Hkv, d, 8, 64, B, 1210, seed=9370 + B)
    for call, inside in ((pod.CALL_ATTENTION, False), (pod.CALL_STEP, True)):
        pl = c.launched(lens, call)
        assert pl["even"] and pl["merge_inside"] == inside, pl
    one = Case(2, 2, Hq, Hkv, d, 8, 64, B, 1210, seed=9370 + B)              # (the oracle wants a token in each: its reference for the others)
    fill_all(c, lens)
    fill_all(one, [max(n, 1) for n in lens])
    for _ in range(2):
        for layer in range(2):
            got = c.decode(layer, lens, max_context_len=max(lens))
            assert float(got[empty].float().abs().max()) == 0.0
            assert_close(got[held], one.decode_ref(layer, [max(n, 1) for n in lens])[held], f"empty sequences, layer {layer}")
    for s in range(2):
        pos = [n + s for n in lens]
        for layer in range(2):
            assert_close(c.step(layer, pos), c.decode_ref(layer, [p + 1 for p in pos]), f"step {s} layer {layer}")
    ctx = [n + 2 for n in lens]
    for layer in range(2):
        assert_close(c.decode(layer, ctx), c.decode_ref(layer, ctx), f"decode layer {layer}")
        for b in empty + held[:2]:
            c.assert_cache_equal(layer, b)
    c.gpu.pod_cache_check()


@pytest.mark.parametrize("d,Hq,inside", [(64, 16, True), (128, 16, True), (64, 56, False), (128, 56, False)])
def test_the_trace_holds_the_walking_workgroups_of_the_launched_split(d, Hq, inside):
    """Steps merged inside and by the second launch: one record per workgroup of pod_decode_even_launch's split, none for the
    workgroups that only take the new token."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    lens = [130 + (91 * i * i) % 900 for i in range(44)] if inside else [2500 + (91 * i * i) % 9000 for i in range(12)]
    c = Case(2, 2, Hq, 4, d, 8, 64, len(lens), max(lens) + 8, seed=9380 + d)
    pl = c.launched(lens, pod.CALL_STEP)
    assert pl["even"] and pl["merge_inside"] == inside, pl
    fill_all(c, lens)
    split = pod.pod_decode_even_launch(cus, 4, 72, lens)
    assert cus != 256 or split["padded"]
    trace = torch.zeros(8 * 2048, dtype=torch.int64, device=c.dev)
    c.gpu.pod_profile_set_trace(trace)
    out = c.step(0, lens)
    c.gpu.pod_profile_set_trace(None)
    assert_close(out, c.decode_ref(0, [n + 1 for n in lens]), f"d={d}")
    words = trace.view(-1, 8).cpu()
    n = split["workgroups"]
    assert (words[:n, 0] == torch.arange(n)).all() and (words[:n, 6] >= words[:n, 2]).all() and (words[:n, 2] > 0).all()
    assert (words[n:] == 0).all()


def test_wrong_context_length_is_flagged_in_the_even_split(monkeypatch):
    monkeypatch.setenv("POD_DECODE_FUSED", "0")
    lens = [900, 300, 77]
    c = Case(2, 2, 4, 2, 64, 8, 32, 3, 1000, seed=9400)
    fill_all(c, lens)
    q = c.decode_queries(0, lens, c.dev)
    ctx = torch.tensor([900, 299, 77], dtype=torch.int32, device=c.dev)      # sequence 1 holds 300
    out = c.gpu.pod_decode_attention(0, q, None, ctx, c.scale)
    with pytest.raises(pod.PodError) as e:
        c.gpu.pod_cache_check()
    assert e.value.code == pod.binding.ERR_STATE
    assert float(out[1].float().abs().max()) == 0.0
    ref = c.decode_ref(0, lens)
    assert_close(out[[0, 2]], ref[[0, 2]], "the other sequences")


@pytest.mark.parametrize("rounds", ["one-round", "several-rounds"])
def test_walk_direction_does_not_change_the_result(rounds, monkeypatch):
    """The layers of a block walk the block's distant keys in alternating directions; with every layer walking forward
    (POD_DECODE_WALK_TURNS=0) the outputs differ only by the order of the sums.  G = 3: forward, backward, forward."""
    outs = {}
    lens = [2500, 700, 90]
    for turns in ("1", "0"):
        monkeypatch.setenv("POD_DECODE_WALK_TURNS", turns)
        if rounds == "several-rounds":
            monkeypatch.setenv("POD_DECODE_FUSED", "0")
        c = Case(3, 3, 8, 2, 128, 8, 64, len(lens), 2600, seed=9700, with_oracle_cache=(turns == "1"))
        fill_all(c, lens)
        o = []
        for s in range(2):
            pos = [n + s for n in lens]
            for layer in range(3):
                out = c.step(layer, pos)
                if turns == "1":
                    assert_close(out, c.decode_ref(layer, [p + 1 for p in pos]), f"step {s} layer {layer}")
                o.append(out.float())
        ctx = [n + 2 for n in lens]
        o += [c.decode(layer, ctx).float() for layer in range(3)]
        outs[turns] = o
        c.gpu.pod_cache_check()
    for a, b in zip(outs["1"], outs["0"]):
        assert (a - b).abs().max() <= 2.0 ** -7 * b.abs().max()


EVEN, EVEN2, FIXED = (True, True), (True, False), (False, True) # (the even split, merged inside)


@pytest.mark.parametrize("d,Hq,Hkv,B,lo,hi,attention,step", [
    (128, 32, 8, 18, 59, 592, EVEN, EVEN),       # more slots than CUs, merged inside
    (128, 32, 4, 70, 40, 200, EVEN, EVEN),       # ... with 8 query heads per kv head
    (128, 64, 4, 68, 60, 80, EVEN, EVEN),        # ... with 16
    (128, 4, 4, 66, 60, 220, EVEN, EVEN),        # ... with one
    (128, 32, 4, 18, 93, 938, FIXED, FIXED),     # fewer slots than CUs
    (128, 32, 4, 3, 3000, 30000, FIXED, EVEN2),  # lengths that fill half of the slots; many partials of 8 query heads
    (128, 32, 4, 3, 900, 9000, FIXED, FIXED),
    (128, 32, 8, 7, 500, 5000, EVEN, EVEN),
    (128, 16, 1, 2, 9000, 12000, EVEN2, EVEN2),  # 16 query heads and more than 16 partials of few pairs
    (64, 16, 4, 5, 700, 7000, EVEN, EVEN),
    (64, 8, 8, 11, 200, 900, EVEN, EVEN),        # no room for the steps' own workgroups
    (64, 64, 8, 8, 200, 900, FIXED, EVEN)])
def test_launches_that_leave_the_fixed_pieces(d, Hq, Hkv, B, lo, hi, attention, step):
    """Ragged batches and shapes on both sides of each rule where the even split takes over from fixed pieces merged inside one round:
    plain decode (one empty sequence among them at the end) and steps against the oracle."""
    S, W = 16, 240
    lens = [lo + (i * 7919) % (hi - lo + 1) for i in range(B)]
    lens[-1] = hi
    c = Case(2, 2, Hq, Hkv, d, S, W, B, hi + 8, seed=590 + B)
    for call, want in ((pod.CALL_ATTENTION, attention), (pod.CALL_STEP, step)):
        pl = c.launched(lens, call)
        assert (pl["even"], pl["merge_inside"]) == want, pl
    for layer in range(2):
        for b, n in enumerate(lens):
            c.fill(layer, b, n)
    for layer in range(2):
        assert_close(c.decode(layer, lens), c.decode_ref(layer, lens), f"decode layer {layer}")
    for s in range(2):
        pos = [n + s for n in lens]
        for layer in range(2):
            assert_close(c.step(layer, pos), c.decode_ref(layer, [p + 1 for p in pos]), f"step {s} layer {layer}")
    ctx = [n + 2 for n in lens[:-1]] + [0]
    out = c.decode(1, ctx)
    assert float(out[-1].float().abs().max()) == 0.0
    for b in (0, B - 1):
        c.assert_cache_equal(0, b)
        c.assert_cache_equal(1, b)

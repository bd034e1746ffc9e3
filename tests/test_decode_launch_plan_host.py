"""How a decode call is launched (host logic, no GPU): pod_decode_launch_plan, the choice that pod_launch_decode makes."""
import numpy as np
import pytest

import paper_2412_02252_amd as pod

CUS, XCDS = 256, 8


def launch(Hq, Hkv, d, P, lens, call=pod.CALL_STEP, **kw):
    return pod.pod_decode_launch_plan(CUS, XCDS, Hq, Hkv, d, P, lens, call, **kw)


def form(pl):
    return ("even" if pl["even"] else "fixed", "inside" if pl["merge_inside"] else "second launch", pl["waves"])


@pytest.mark.parametrize("seed", range(40))
def test_the_choice_agrees_with_the_plans_it_is_made_of(seed):
    """Fixed pieces of eight waves are pod_decode_plan's, the even split is pod_decode_even_launch's; who merges, who hands over inside one XCD and
    which scratch suffices follow from that."""
    rng = np.random.default_rng(8100 + seed)
    for _ in range(60):
        Hkv, rep, d = int(rng.choice([1, 2, 3, 4, 8, 16])), int(rng.choice([1, 2, 4, 5, 8, 16])), int(rng.choice([64, 128]))
        P, B = int(rng.choice([40, 272, 2112])), int(rng.choice([1, 1, 2, 3, 8, 17, 40, 200]))
        hi = int(2 ** rng.uniform(0, 17))
        lens = [int(x) for x in rng.integers(max(0, int(hi * rng.choice([0, 0.1, 0.9]))), hi + 1, size=B)]
        call, known = int(rng.integers(0, 4)), bool(rng.integers(0, 8))
        pl = launch(Hkv * rep, Hkv, d, P, lens, call, lens_known=known)
        what = (Hkv, rep, d, P, lens, call, known, pl)
        step, bound = call != pod.CALL_ATTENTION, max(max(lens) + (call != pod.CALL_ATTENTION), 1)
        plain = call in (pod.CALL_ATTENTION, pod.CALL_STEP)
        fixed = pod.pod_decode_plan(CUS, B, Hkv, P, bound)
        if pl["even"]:
            ev = pod.pod_decode_even_launch(CUS, Hkv, P, lens, 128 if plain else 256)
            assert known and call != pod.CALL_REUSE_FIRST and pl["waves"] == 4 and not pl["xcd_local"], what
            assert pl["units_per_workgroup"] == ev["units_per_workgroup"] and pl["partials"] == ev["partials_per_pair"] + step, what
            assert pl["padded"] == ev["padded"] and pl["own_workgroup"] == step, what
            assert not pl["merge_inside"] or (pl["padded"] and plain and (step or min(lens) > 0)), what
            # in less scratch than its partials take the launch keeps to fixed pieces
            need = B * Hkv * rep * pl["partials"] * (d + 2) * 4
            assert launch(Hkv * rep, Hkv, d, P, lens, call, workspace_bytes=need)["even"]
            assert not launch(Hkv * rep, Hkv, d, P, lens, call, workspace_bytes=need - 1)["even"]
        else:
            pieces = pl["partials"] - step
            assert pl["merge_inside"] or not (pl["xcd_local"] or pl["own_workgroup"] or pl["waves"] == 8), what
            assert step or not pl["own_workgroup"], what
            if pl["waves"] == 8 and plain:
                assert fixed["merge_inside"] and (pl["chunk"], pl["chunk_prox"], pieces) == (fixed["chunk"], fixed["chunk_prox"], fixed["pieces"]), what
            if pl["waves"] == 4 and pl["merge_inside"]: # a small launch: a CU for each of an XCD's workgroups
                assert pl["xcd_local"] and -(-B * Hkv // XCDS) * pl["partials"] <= CUS // XCDS, what
                assert pl["own_workgroup"] == step, what # (score reuse's kernel of four waves has one as a constant)
            if pl["own_workgroup"]:
                assert B * Hkv * pl["partials"] <= (-(-B * Hkv // XCDS) * XCDS * (CUS // XCDS) if pl["xcd_local"] else CUS), what


def test_forms_of_usual_calls():
    chats = [300 + 122 * i for i in range(28)]
    assert form(launch(4, 2, 64, 272, [2048])) == ("fixed", "inside", 4)
    assert form(launch(32, 8, 128, 2112, [32768])) == ("fixed", "inside", 8)
    assert form(launch(16, 4, 64, 528, chats)) == ("even", "inside", 4)
    assert form(launch(32, 8, 128, 2112, [4000 + 1800 * i for i in range(16)])) == ("even", "second launch", 4)
    assert form(launch(32, 8, 128, 2112, [32768], pod.CALL_REUSE_FIRST)) == ("fixed", "inside", 8)
    assert form(launch(32, 8, 128, 4224, [131072] * 4, pod.CALL_REUSE_FIRST)) == ("fixed", "second launch", 4)
    assert form(launch(32, 8, 128, 4224, [131072] * 4, pod.CALL_REUSE_UPPER)) == ("even", "second launch", 4)
    assert form(launch(16, 4, 64, 528, chats, lens_known=False)) == ("fixed", "second launch", 4)


@pytest.mark.parametrize("d,Hq,Hkv,call,n,waves", [
    (128, 32, 8, pod.CALL_ATTENTION, 1000, 4),  # 8 pieces: attention keeps no row for a step ...
    (128, 32, 8, pod.CALL_STEP, 1000, 8),       # ... and a step has 9
    (128, 32, 8, pod.CALL_ATTENTION, 1025, 8),  # 9 pieces
    (64, 40, 5, pod.CALL_ATTENTION, 1000, 4),   # 8 rows: any number of query heads
    (64, 40, 5, pod.CALL_ATTENTION, 2493, 8),   # 20 rows, 8 query heads per kv head: eight waves merge them sooner
    (64, 16, 1, pod.CALL_STEP, 2007, 8),
    (64, 6, 1, pod.CALL_REUSE_FIRST, 2007, 8),
    (64, 16, 4, pod.CALL_STEP, 2493, 4),        # four: sooner than eight waves' 11 rows
    (64, 16, 4, pod.CALL_STEP, 1500, 8),        # eight waves leave 7
    (64, 4, 2, pod.CALL_STEP, 1500, 4),
])
def test_which_small_launches_run_workgroups_of_four_waves(d, Hq, Hkv, call, n, waves):
    pl = launch(Hq, Hkv, d, 256, [n], call)
    assert form(pl) == ("fixed", "inside", waves), pl


@pytest.mark.parametrize("d,Hq,Hkv,lens,partials,inside", [ # partials per query head, without a step's
    (128, 32, 8, [131072], 61, False),         # 4 x 61: one workgroup would merge 244
    (128, 32, 8, [65536] * 2, 31, True),       # 4 x 31
    (128, 16, 8, [131072], 61, True),          # 2 x 61
    (128, 4, 1, [1000000], 489, False),
    (128, 1, 1, [1000000], 489, False),        # one query head, but a chain of 489
    (64, 32, 8, [131072], 61, True),           # head dimension 64: 4 x 62
    (64, 32, 8, [88826], 64, True),            # 4 x 65, a whole chip's share for eight kv heads and a step's own
    (64, 16, 4, [300000], 124, False),
    (128, 32, 4, [600 + 20 * i for i in range(36)], 4, True),      # 8 x 4
    (128, 32, 4, [40000] * 4, 32, False),      # 8 x 32
    (128, 64, 4, [900 + 10 * i for i in range(40)], 3, True),      # 16 x 3
    (128, 16, 1, [30000, 16000], 236, False),
])
def test_the_even_split_merges_inside_where_one_workgroup_has_few_partials(d, Hq, Hkv, lens, partials, inside):
    for call in (pod.CALL_ATTENTION, pod.CALL_STEP):
        pl = launch(Hq, Hkv, d, 272, lens, call)
        assert pl["even"] and pl["padded"] and pl["partials"] == partials + (call == pod.CALL_STEP), pl
        assert pl["merge_inside"] == inside, pl


@pytest.mark.parametrize("d,Hq,Hkv,P,lens,call,want", [
    # more pieces than CUs
    (128, 32, 8, 272, [59 + 31 * i for i in range(18)], pod.CALL_STEP, "even inside"),
    (128, 64, 4, 528, [71] * 68, pod.CALL_STEP, "even inside"),
    (128, 64, 4, 528, [210 + i * 204 // 78 for i in range(79)], pod.CALL_STEP, "fixed"),     # a second launch for short pairs costs more
    (128, 64, 4, 4224, [1976] * 71, pod.CALL_STEP, "even second launch"),
    (64, 128, 8, 4224, [400 + i * 11 for i in range(34)], pod.CALL_STEP, "even second launch"),
    (128, 64, 8, 2112, [10940, 17000, 23853], pod.CALL_ATTENTION, "fixed"),
    # many partials of few pairs with sixteen query heads
    (128, 16, 1, 272, [14000, 27000], pod.CALL_STEP, "even second launch"),
    (64, 16, 1, 272, [4856] * 4, pod.CALL_STEP, "fixed"),
    (64, 16, 1, 4224, [12856, 13977], pod.CALL_STEP, "even second launch"),
    # lengths that differ, merged inside and by a second launch
    (128, 32, 8, 272, [500, 800, 1200, 2000, 3000, 4000, 5000], pod.CALL_STEP, "even inside"),
    (128, 32, 8, 272, [5502 + 80 * i for i in range(7)] + [6085], pod.CALL_STEP, "fixed"),
    (64, 16, 4, 528, [700, 1500, 2500, 4000, 12000], pod.CALL_STEP, "even inside"),
    (64, 16, 4, 2112, [3691, 21823], pod.CALL_STEP, "fixed"),
    (64, 8, 8, 272, [1159] * 16, pod.CALL_ATTENTION, "fixed"),
    # long pieces, and steps without room for their own workgroups, at head dimension 64
    (64, 16, 4, 528, [19000] * 4, pod.CALL_STEP, "even inside"),
    (64, 16, 2, 1004, [33661] * 7, pod.CALL_ATTENTION, "fixed"),
    (64, 16, 4, 528, [600 + 60 * i for i in range(11)], pod.CALL_STEP, "even inside"),
    (64, 64, 8, 272, [457 + 60 * i for i in range(8)], pod.CALL_STEP, "even inside"),
    (64, 256, 16, 528, [1087] * 3, pod.CALL_STEP, "fixed"),
])
def test_launches_of_one_round_that_leave_the_fixed_pieces(d, Hq, Hkv, P, lens, call, want):
    """Each rule on the side where the even split ends sooner and on the one where fixed pieces do."""
    assert pod.pod_decode_plan(CUS, len(lens), Hkv, P, max(lens) + (call == pod.CALL_STEP))["merge_inside"]
    pl = launch(Hq, Hkv, d, P, lens, call)
    assert " ".join(form(pl)[:2]) == ("fixed inside" if want == "fixed" else want), pl


def test_bad_arguments_are_rejected():
    good = dict(num_cus=CUS, num_xcds=XCDS, num_q_heads=8, num_kv_heads=2, head_dim=64, proximal_rows=72, context_lens=[100])
    pod.pod_decode_launch_plan(**good)
    for bad in (dict(num_cus=0), dict(num_xcds=-1), dict(num_q_heads=7), dict(num_q_heads=34), dict(num_kv_heads=0), dict(head_dim=96),
                dict(proximal_rows=0), dict(call=4), dict(call=-1), dict(max_context_len=-1), dict(context_lens=[100] * 257)):
        with pytest.raises(pod.PodError) as e:
            pod.pod_decode_launch_plan(**{**good, **bad})
        assert e.value.code == pod.binding.ERR_INVALID_ARG


def test_a_launch_that_keeps_fixed_pieces_is_chosen_without_planning_the_even_split():
    """250 pairs of one short piece each: the split of such a batch costs the host more than everything else of the choice."""
    import ctypes as C
    import time
    L, B = pod.load(), 250
    lens, plan, cum = (C.c_int32 * B)(*[100] * B), (C.c_int32 * 8)(), (C.c_int32 * (B + 1))()

    def fastest(call):
        best = float("inf")
        for _ in range(100):
            t0 = time.perf_counter()
            for _ in range(20):
                assert call() == 0
            best = min(best, time.perf_counter() - t0)
        return best / 20

    choice = lambda known: fastest(lambda: L.pod_decode_launch_plan(CUS, XCDS, B, 8, 1, 128, 272, 101, lens if known else None, pod.CALL_STEP, 1 << 30, plan))
    split = fastest(lambda: L.pod_decode_even_launch(CUS, B, 1, 272, 128, lens, plan, cum)) - fastest(lambda: L.pod_decode_even_launch(CUS, 1, 1, 272, 128, lens, plan, cum))
    assert not launch(8, 1, 128, 272, [100] * B)["even"]
    assert choice(True) - choice(False) < 0.5 * split, (choice(True), choice(False), split)

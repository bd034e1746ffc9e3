"""GPU: head-wise blocks (a table lowest[layer][kv head] instead of uniform blocks) against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_2412_02252_amd as pod
from oracle import pod_oracle as po
from pod_inputs import gen
from podcase import Case, assert_close

pytestmark = pytest.mark.gpu

# kv head 0: one block of all four layers; head 1: {0,1},{2,3}; head 2: every layer alone
MAP4 = np.array([[0, 0, 0], [0, 0, 1], [0, 2, 2], [0, 2, 3]], dtype=np.int32)


def gathered(c, layer, what, seq, n, device):
    """k_shared [n][Hkv][d] or q_shared [n][Hq][d] for a prompt: head by head from the lowest layer of its block."""
    src = c.lowest[layer]
    rep = c.Hq // c.Hkv
    if what == "k":
        per = {int(l): c.keys(int(l), seq, n, device) for l in set(src.tolist())}
        return torch.stack([per[int(src[h])][:, h] for h in range(c.Hkv)], dim=1).contiguous()
    per = {int(l): c.queries(int(l), seq, n, device) for l in set(src.tolist())}
    return torch.stack([per[int(src[h // rep])][:, h] for h in range(c.Hq)], dim=1).contiguous()


@pytest.mark.parametrize("d", [128, 64])
def test_cache_and_decode_with_a_headwise_table(d):
    L, Hq, Hkv, S, W = 4, 6, 3, 8, 32
    lens = [150, 41, 300]
    c = Case(L, 1, Hq, Hkv, d, S, W, len(lens), 400, seed=700 + d, block_lowest=MAP4)
    for layer in range(L):
        for b, n in enumerate(lens):
            c.fill(layer, b, n)
    for step in range(3):                                   # appends with demotion, every layer in step
        pos = [n + step for n in lens]
        for layer in range(L):
            c.append(layer, pos)
        ctx = [p + 1 for p in pos]
        for layer in range(L):
            assert_close(c.decode(layer, ctx), c.decode_ref(layer, ctx), f"step {step} layer {layer}")
    for layer in range(L):
        for b in range(len(lens)):
            c.assert_cache_equal(layer, b)                  # incl. distant keys only where the layer is a head's lowest
    c.gpu.pod_cache_check()
    live, _ = pod.pod_cache_live_bytes(c.cfg, 1)            # (sizes are per sequence)
    assert c.cpu.stored_elems() * 2 == sum(pod.pod_cache_live_bytes(c.cfg, n + 3)[0] for n in lens)


def test_prefill_with_a_headwise_table():
    L, Hq, Hkv, d, S, W, n = 4, 6, 3, 128, 8, 40, 333
    c = Case(L, 1, Hq, Hkv, d, S, W, 1, 600, seed=711, block_lowest=MAP4)
    rows = np.arange(n)
    for layer in range(L):
        q, k, v = c.queries(layer, 0, n, c.dev), c.keys(layer, 0, n, c.dev), c.values(layer, 0, n, c.dev)
        all_lowest = bool((c.lowest[layer] == layer).all())
        qs = None if all_lowest else gathered(c, layer, "q", 0, n, c.dev)
        ks = None if all_lowest else gathered(c, layer, "k", 0, n, c.dev)
        out = c.gpu.pod_prefill_attention(layer, 0, q, k, v, qs, ks, c.scale, write_cache=True)
        qc = gen.bf16_bits(c.queries(layer, 0, n, "cpu"))
        kc, vc = gen.bf16_bits(c.keys(layer, 0, n, "cpu")), gen.bf16_bits(c.values(layer, 0, n, "cpu"))
        qsc = None if all_lowest else gen.bf16_bits(gathered(c, layer, "q", 0, n, "cpu"))
        ksc = None if all_lowest else gen.bf16_bits(gathered(c, layer, "k", 0, n, "cpu"))
        assert_close(out, po.pod_attention(qc, kc, vc, qsc, ksc, rows, S, W, c.scale), f"layer {layer}")
        c.cpu.fill(layer, 0, kc, vc)
        c.assert_cache_equal(layer, 0)
    # the cache prefill built serves decode
    for layer in range(L):
        c.append(layer, [n])
    for layer in range(L):
        assert_close(c.decode(layer, [n + 1]), c.decode_ref(layer, [n + 1]), f"decode layer {layer}")
    c.gpu.pod_cache_check()


def test_explicit_uniform_table_behaves_like_group_size():
    L, G, Hq, Hkv, d, S, W, n = 4, 2, 8, 2, 128, 8, 32, 200
    uni = np.array([[l - l % G] * Hkv for l in range(L)], dtype=np.int32)
    a = Case(L, G, Hq, Hkv, d, S, W, 1, 300, seed=720)
    b = Case(L, 1, Hq, Hkv, d, S, W, 1, 300, seed=720, block_lowest=uni)
    for layer in range(L):
        a.fill(layer, 0, n)
        b.fill(layer, 0, n)
    for layer in range(L):
        assert torch.equal(a.decode(layer, [n]), b.decode(layer, [n]))
    scores = b.gpu.new_score_buffer()                       # a uniform table also allows score reuse
    for layer in range(L):
        assert_close(b.decode_reuse(layer, [n], scores), b.decode_ref(layer, [n]), f"reuse layer {layer}")


def test_lagging_lowest_layer_of_one_head_is_caught_on_the_host():
    c = Case(4, 1, 6, 3, 64, 8, 32, 1, 300, seed=730, block_lowest=MAP4)
    for layer in range(4):
        c.fill(layer, 0, 100)
    # layer 3 moves ahead of layer 2, the lowest layer of kv head 1's block: refused on the host
    c.append(3, [100])
    with pytest.raises(pod.PodError) as e:
        c.decode(3, [101])
    assert e.value.code == pod.binding.ERR_STATE


@pytest.mark.parametrize("d", [128, 64])
def test_score_reuse_with_a_headwise_table(d):
    """Layers in ascending order through the score-reuse entry point: at each layer the kv heads whose block
    starts there write their logits, the others read theirs (MAP4 has layers that do both at once)."""
    L, Hq, Hkv, S, W = 4, 6, 3, 8, 32
    lens = [150, 41, 300]
    c = Case(L, 1, Hq, Hkv, d, S, W, len(lens), 400, seed=740 + d, block_lowest=MAP4)
    for layer in range(L):
        for b, n in enumerate(lens):
            c.fill(layer, b, n)
    scores = c.gpu.new_score_buffer()
    for step in range(2):
        pos = [n + step for n in lens]
        for layer in range(L):
            c.append(layer, pos)
        ctx = [p + 1 for p in pos]
        for layer in range(L):
            assert_close(c.decode_reuse(layer, ctx, scores), c.decode_ref(layer, ctx), f"step {step} layer {layer}")
    c.gpu.pod_cache_check()
    # a stale buffer: layer 3 reads head 1's logits of the previous token -> rows zeroed, flag raised
    pos = [n + 2 for n in lens]
    for layer in range(L):
        c.append(layer, pos)
    ctx = [p + 1 for p in pos]
    out = c.decode_reuse(3, ctx, scores)
    with pytest.raises(pod.PodError):
        c.gpu.pod_cache_check()
    rep = Hq // Hkv                                         # (sequence 1 has no distant tokens: nothing to check there)
    assert float(out[0, : 2 * rep].float().abs().max()) == 0.0     # kv heads 0 and 1 read stale logits at layer 3
    assert_close(out[0, 2 * rep:], c.decode_ref(3, ctx)[0, 2 * rep:], "kv head 2 starts a block at layer 3: exact")


def test_gated_skip_with_a_headwise_table():
    """Per head: no gate where the layer is the lowest of the head's block, the gate of Eq. 4 elsewhere;
    decisions and outputs against the oracle for tau = 1 (never), 0 (always) and a value between the gates."""
    L, Hq, Hkv, d, S, W = 4, 6, 3, 128, 8, 64
    lens = [500, 260]
    c = Case(L, 1, Hq, Hkv, d, S, W, len(lens), 600, seed=750, block_lowest=MAP4)
    for layer in range(L):
        for b, n in enumerate(lens):
            c.fill(layer, b, n)
    scores = c.gpu.new_score_buffer()
    ctx_t = torch.tensor(lens, dtype=torch.int32, device=c.dev)

    def both(layer, tau):
        got = c.gpu.pod_decode_attention_gated(layer, c.decode_queries(layer, lens, c.dev), ctx_t, c.scale, tau, scores)
        flags = c.gpu.skip_flags(scores)[: len(lens)].cpu().numpy().copy()
        qs = c.shared_queries(layer, lens, "cpu")
        ref, g, skipped = c.cpu.decode_attention_gated(layer, gen.bf16_bits(c.decode_queries(layer, lens, "cpu")),
                                                       gen.bf16_bits(qs) if qs is not None else None, lens, c.scale, tau)
        return got, flags, ref, g, skipped

    rep = Hq // Hkv
    for tau in (1.0, 0.0, None):
        for layer in range(L):
            if tau is None:                                  # a threshold inside the widest gap of this layer's gates
                _, _, _, g, _ = both(layer, 1.0)
                upper = np.repeat(c.lowest[layer] != layer, rep)
                gs = np.sort(g[:, upper].ravel())
                if len(gs) < 2:
                    t = 0.5
                else:
                    gaps = np.diff(gs)
                    t = float(gs[np.argmax(gaps)] + gaps.max() / 2)
                    if gaps.max() < 0.04:
                        t = 0.0
            else:
                t = tau
            got, flags, ref, g, skipped = both(layer, t)
            upper = np.repeat(c.lowest[layer] != layer, rep)
            np.testing.assert_array_equal(flags[:, upper], skipped[:, upper], err_msg=f"tau={t} layer {layer}")
            assert not skipped[:, ~upper].any()              # heads for which the layer is the lowest never skip
            assert_close(got, ref, f"tau={t} layer {layer}")
    c.gpu.pod_cache_check()


# ---------------------------------------------------------------- attention similarity -> grouping -> table

from oracle import pod_grouping as pg


@pytest.mark.parametrize("L,H,R,n", [(3, 2, 4, 64), (5, 4, 6, 1000), (2, 1, 1, 4), (4, 3, 3, 4100), (19, 2, 2, 514), (32, 1, 2, 1024),
                                     (8, 2, 1, 8), (9, 1, 4, 333),
                                     # enough workgroups for blocks of four layers; 18 heads do not deal out over 8 XCDs
                                     (32, 8, 3, 68), (19, 18, 2, 34)])
def test_layer_similarity_matches_the_oracle(L, H, R, n):
    rng = np.random.default_rng(L * 1000 + n)
    att = rng.dirichlet(np.full(n, 0.3), size=(L, H, R)).astype(np.float32)
    att[0, 0, 0, : n // 2] = 0                               # exact zeros: 0 log 0 = 0
    att[0, 0, 0, n // 2] = 1e-41                             # and a subnormal entry
    att[0, 0, 0] /= att[0, 0, 0].sum()
    if L > 1:
        att[1] = att[0]                                      # two identical layers: similarity exactly 1
    got = pod.pod_layer_similarity(torch.from_numpy(att).cuda()).cpu().numpy()
    ref = np.ones((H, L, L))
    for h in range(H):
        for a in range(L):
            for b in range(a + 1, L):
                ref[h, a, b] = ref[h, b, a] = pg.layer_similarity(att[a, h][None], att[b, h][None])
    np.testing.assert_allclose(got, ref, rtol=0, atol=2e-5)  # fp32 sums of up to 25000 terms of size <= 1
    if L > 1:
        assert np.abs(got[:, 0, 1] - 1).max() < 1e-6
    assert (got >= -1e-6).all() and (got <= 1 + 1e-6).all()


@pytest.mark.parametrize("L,H,R,n,streamed", [(29, 16, 1, 2052, 4), (30, 16, 2, 34, 4), (31, 32, 1, 4, 4), (32, 32, 1, 8, 4), (13, 32, 3, 68, 4),
                                              (29, 16, 1, 20004, 8), (30, 32, 1, 10004, 8), (31, 32, 3, 3404, 8), (32, 32, 2, 5000, 8), (45, 32, 1, 4444, 8)])
def test_layer_similarity_in_blocks_of_four_by_four_and_by_eight(L, H, R, n, streamed):
    """Block pairs of 4 x 4 and (on 256 CUs) 4 x 8 layers: the last block of eight whole, or with one to three layers in its second half;
    elements for one thread only, and for every thread more than once."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus != 256 or pod.pod_similarity_plan(cus, L, H, R, n) == (4, streamed)
    gen = torch.Generator(device="cuda").manual_seed(L * 100 + n)
    att = torch.softmax(3 * torch.randn((L, H, R, n), generator=gen, device="cuda"), -1).contiguous()
    att[L - 1] = att[2]
    got = pod.pod_layer_similarity(att)
    for h in range(H):
        x = att[:, h].double()
        e = torch.special.xlogy(x, x).sum((1, 2))
        for a in range(L):
            m = 0.5 * (x[a] + x)
            ref = 1 - (0.5 * (e[a] + e) - torch.special.xlogy(m, m).sum((1, 2))) / (R * np.log(2.0))
            ref[a] = 1
            assert (got[h, a].double() - ref).abs().max() < 2e-6, (h, a)      # fp32 sums of terms that add up to at most 1
    assert (got[:, 2, L - 1] == 1).all() and (got[:, L - 1, 2] == 1).all()


@pytest.mark.parametrize("L,H,n", [(2, 400, 4), (8, 64, 8), (32, 40, 60), (3, 100, 256)])
def test_layers_with_the_same_rows_have_similarity_one_exactly(L, H, n):
    """One sampled row per head, so that no average rounds a remainder away; blocks of two and of four layers.  A threshold of 1
    groups such layers."""
    rng = np.random.default_rng(L * 1000 + n)
    att = rng.dirichlet(np.full(n, 0.3), size=(L, H, 1)).astype(np.float32)
    att[L - 1] = att[0]
    att[1, : H // 2] = att[0, : H // 2]
    got = pod.pod_layer_similarity(torch.from_numpy(att).cuda()).cpu().numpy()
    assert (got[:, 0, L - 1] == 1).all() and (got[:, L - 1, 0] == 1).all()
    assert (got[: H // 2, 0, 1] == 1).all()
    lowest = pod.pod_group_layers(got[: H // 2, [0, 1]][:, :, [0, 1]], H // 2, 1.0)
    assert (np.asarray(lowest) == 0).all()


def test_layer_similarity_of_more_workgroups_than_a_grid_dimension_holds():
    """512 layers x 1024 heads: 8256 pairs of four-layer blocks, in two halves per head, are 2^32 threads and more.  Every value is
    compared."""
    L, H, n = 512, 1024, 4
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    att = torch.softmax(torch.randn((L, H, 1, n), generator=gen, device="cuda"), -1).contiguous()
    got = pod.pod_layer_similarity(att)
    for h in range(H):
        x = att[:, h, 0].double()
        e, m = torch.special.xlogy(x, x).sum(1), 0.5 * (x[:, None] + x[None])
        ref = 1 - (0.5 * (e[:, None] + e[None]) - torch.special.xlogy(m, m).sum(2)) / np.log(2.0)
        assert (got[h].double() - ref).abs().max() < 2e-6, h      # four terms below 1 in fp32


def test_similarity_to_grouping_to_cache_table():
    """Layers 0-2 share one attention pattern, layers 3-4 another (plus noise), per head differently:
    the GPU similarity, the host grouping and a cache built from the table agree with the oracle chain."""
    rng = np.random.default_rng(99)
    L, Hq, Hkv, R, n = 5, 4, 2, 8, 256
    base = rng.dirichlet(np.full(n, 0.1), size=(2, Hq, R))
    att = np.empty((L, Hq, R, n), np.float32)
    for l in range(L):
        for h in range(Hq):
            pattern = 0 if (l < 3 if h < 2 else l < 2) else 1   # heads 0,1 split after layer 2; heads 2,3 after layer 1
            noisy = base[pattern, h] * rng.uniform(0.9, 1.1, size=(R, n))
            att[l, h] = noisy / noisy.sum(axis=1, keepdims=True)
    sim = pod.pod_layer_similarity(torch.from_numpy(att).cuda()).cpu().numpy()
    table = pod.pod_group_layers(sim, Hkv, 0.5)
    sim_ref = np.ones((Hq, L, L))
    for h in range(Hq):
        for a in range(L):
            for b in range(a + 1, L):
                sim_ref[h, a, b] = sim_ref[h, b, a] = pg.layer_similarity(att[a, h][None], att[b, h][None])
    np.testing.assert_array_equal(table, pg.group_layers_gqa(sim_ref, Hkv, 0.5))
    assert table[:, 0].tolist() == [0, 0, 0, 3, 3] and table[:, 1].tolist() == [0, 0, 2, 2, 2]
    c = Case(L, 1, Hq, Hkv, 64, 8, 32, 1, 200, seed=750, block_lowest=table)
    for layer in range(L):
        c.fill(layer, 0, 150)
    for layer in range(L):
        assert_close(c.decode(layer, [150]), c.decode_ref(layer, [150]), f"layer {layer}")

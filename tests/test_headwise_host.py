"""CPU: host logic for head-wise blocks in libpod (layer grouping, sizes, table validation) against the oracle."""
import ctypes as C

import numpy as np
import pytest

import paper_2412_02252_amd as pod
from oracle import pod_grouping as pg
from oracle import pod_oracle as po

MAP4 = np.array([[0, 0, 0], [0, 0, 1], [0, 2, 2], [0, 2, 3]], dtype=np.int32)


@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (8, 2), (12, 4), (6, 2)])
def test_group_layers_matches_the_oracle_on_random_similarities(Hq, Hkv):
    rng = np.random.default_rng(7 * Hq + Hkv)
    for trial in range(20):
        L = int(rng.integers(1, 12))
        sim = rng.random((Hq, L, L)).astype(np.float32)
        sim = np.maximum(sim, sim.transpose(0, 2, 1))          # symmetric, like a similarity
        thr = float(rng.choice([0.3, 0.5, 0.7]))
        got = pod.pod_group_layers(sim, Hkv, thr)
        want = pg.group_layers_gqa(sim, Hkv, thr)
        np.testing.assert_array_equal(got, want)
        if Hq == Hkv:
            np.testing.assert_array_equal(got, pg.group_layers(sim, thr))


def test_group_layers_output_is_a_valid_block_table():
    rng = np.random.default_rng(3)
    sim = rng.random((8, 16, 16)).astype(np.float32)
    tab = pod.pod_group_layers(sim, 4, 0.5)
    cfg = pod.make_config(16, 1, 8, 4, 64, 4, 8, 1, 64, block_lowest=tab)
    assert pod.pod_cache_bytes(cfg) > 0


def test_sizes_with_a_table_match_the_oracle_formula():
    L, Hq, Hkv, d, S, W, n = 4, 6, 3, 64, 4, 8, 1000
    cfg = pod.make_config(L, 1, Hq, Hkv, d, S, W, 1, 2048, block_lowest=MAP4)
    live, dense = pod.pod_cache_live_bytes(cfg, n)
    assert (live, dense) == tuple(int(x) for x in po.cache_bytes_formula_map(MAP4, d, S, W, n))
    uni = np.array([[l - l % 2] * Hkv for l in range(L)], dtype=np.int32)
    a = pod.make_config(L, 2, Hq, Hkv, d, S, W, 1, 2048)
    b = pod.make_config(L, 1, Hq, Hkv, d, S, W, 1, 2048, block_lowest=uni)
    assert pod.pod_cache_bytes(a) == pod.pod_cache_bytes(b)
    assert pod.pod_cache_live_bytes(a, n) == pod.pod_cache_live_bytes(b, n)
    # 7 (kv head, block) pairs instead of 6 for uniform pairs of layers: one more distant-key store
    extra = pod.pod_cache_bytes(cfg) - pod.pod_cache_bytes(a)
    assert extra == (2048 - S - W) * d * 2


def test_invalid_tables_are_refused():
    bad = MAP4.copy()
    bad[3, 1] = 1
    with pytest.raises(pod.PodError):
        pod.pod_cache_bytes(pod.make_config(4, 1, 6, 3, 64, 4, 8, 1, 64, block_lowest=bad))
    bad = MAP4.copy()
    bad[0, 0] = 1
    with pytest.raises(pod.PodError):
        pod.pod_cache_bytes(pod.make_config(4, 1, 6, 3, 64, 4, 8, 1, 64, block_lowest=bad))
    with pytest.raises(ValueError):
        pod.make_config(4, 1, 6, 3, 64, 4, 8, 1, 64, block_lowest=MAP4[:3])


@pytest.mark.parametrize("layers,heads", [(65536, 1), (1, 65536), (65537, 1), (2, 70000)])
def test_similarity_refuses_what_it_cannot_launch(layers, heads):
    """(Refused from the sizes alone: nothing is read or launched.)"""
    buf = (C.c_float * 16)()
    at = (C.addressof(buf) + 15) // 16 * 16
    assert pod.binding.load().pod_layer_similarity(at, layers, heads, 1, 4, at, None) == pod.binding.ERR_INVALID_ARG


@pytest.mark.parametrize("layers,heads,elements,blocks", [
    (32, 32, 65536, (4, 8)), (32, 32, 12000, (4, 8)), (32, 32, 3072, (4, 4)), (32, 16, 768, (4, 4)), (45, 8, 6000, (4, 4)), (40, 32, 1792, (4, 4)),
    (24, 32, 65536, (4, 4)), (16, 24, 65536, (2, 2)), (2, 1, 4, (2, 2)), (65535, 65535, 1 << 20, (4, 8))])
def test_similarity_blocks_follow_the_work(layers, heads, elements, blocks):
    """Blocks of 4 x 8 layers only where there are enough elements per head for half as many workgroups to pay (256 CUs)."""
    assert pod.pod_similarity_plan(256, layers, heads, 1, elements) == blocks
    for bad in ((0, 2, 2, 1, 4), (256, 0, 2, 1, 4), (256, 2, 65536, 1, 4), (256, 2, 2, 0, 4), (256, 2, 2, 1, 0)):
        with pytest.raises(pod.PodError):
            pod.pod_similarity_plan(*bad)

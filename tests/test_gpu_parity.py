"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle.

Tolerances: attention outputs within max relative error 2e-2 per (row, head)
(bf16 inputs and bf16 P for the second product, fp32 accumulation); scores
within 1e-3 relative plus one smallest normal fp32 number per contributing row
(a weight the GPU flushes to zero);
kept sets, merge plans, token indices and weights bit-exact when selection is
fed the oracle's fp32 scores; merged rows within one bf16 ulp (fp32 vs fp64
averaging before the single rounding); untouched rows bit-exact."""
import os
import re

import numpy as np
import pytest
import torch

import paper_2604_16734_amd as K
from kvp_workload import Segment, Workload, get_workload, layer_inputs, bf16_bits_to_f32, chunk_ranges, f32_to_bf16_bits
from oracle import kvp_oracle as O
from tests import gpu_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# Free-running comparison (nothing re-synchronised): floors below what the workloads give, so
# that they flag a real divergence and not a near-tie decided the other way.
FREE_RUNNING_JACCARD_FLOOR = 0.98       # measured: 1.0 on all three
FREE_RUNNING_OUT_TOL = 2e-2             # measured: 4.6e-3


def _rand_bits(rng, shape, scale=1.0):
    from kvp_workload import f32_to_bf16_bits
    return f32_to_bf16_bits((scale * rng.standard_normal(shape)).astype(np.float32))


def _attention_case(hq, hkv, d, c, n, budget, chunk_max, seed, scale=0.0, n_obs=0, keydiff=False,
                    attention_shape=None, fused=None):
    """One prefill_chunk (or prefill_chunk_proxy with n_obs proxy queries) on a cache preloaded
    with c random entries."""
    rng = np.random.default_rng(seed)
    segs = [Segment(0, 100000, 0)]
    cache = K.Cache(1, hq, hkv, d, budget, chunk_max, segs, merge=False, softmax_scale=scale, device=DEV)
    if attention_shape is not None:
        cache.set_attention_shape(attention_shape)
    if fused is not None:
        cache.set_score_sweep(fused)
    oc = O.LayerCache(hkv, d, budget)
    if c:
        kb0, vb0 = _rand_bits(rng, (c, hkv, d)), _rand_bits(rng, (c, hkv, d))
        oc.compact(0, O.bf16_bits_to_f64(kb0), O.bf16_bits_to_f64(vb0), np.zeros((hkv, c), dtype=np.float32))
        perm = np.stack([rng.permutation(c) for _ in range(hkv)])       # slot order is arbitrary
        oc.idx = np.take_along_axis(oc.idx, perm, axis=1)
        oc.K = np.take_along_axis(oc.K, perm[:, :, None], axis=1)
        oc.V = np.take_along_axis(oc.V, perm[:, :, None], axis=1)
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, c)
    qb, kb, vb = _rand_bits(rng, (n, hq, d)), _rand_bits(rng, (n, hkv, d)), _rand_bits(rng, (n, hkv, d))
    q64, k64, v64 = (O.bf16_bits_to_f64(x) for x in (qb, kb, vb))
    out_ref, scores_ref = oc.attend(c, q64, k64, v64, scale or None)
    if keydiff:
        out = cache.prefill_chunk_keydiff(0, c, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
        scores_ref = oc.keydiff(c, k64, v64)
    elif n_obs:
        ob = _rand_bits(rng, (n_obs, hq, d))
        out = cache.prefill_chunk_proxy(0, c, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb),
                                        U.bits_to_torch(ob))
        scores_ref = oc.proxy(c, O.bf16_bits_to_f64(ob), k64, v64, scale or None)
    else:
        out = cache.prefill_chunk(0, c, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
    err = U.out_rel_err(U.torch_bf16_to_f64(out), out_ref)
    # finish the scores the way the library does: compact with its own scores, then read them
    cache.compact(0)
    return cache, oc, err, scores_ref, (q64, k64, v64)


@pytest.mark.parametrize("hq,hkv,d,c,n,budget,chunk_max", [
    (4, 4, 64, 0, 64, 4096, 64),        # empty cache, pure causal block
    (4, 2, 128, 0, 33, 4096, 64),       # ragged single tile, GQA
    (2, 1, 128, 100, 1, 4096, 64),      # a single row
    (8, 2, 128, 193, 150, 4096, 256),   # cache not tile aligned, ragged rows, several key tiles
    (4, 4, 64, 70, 129, 4096, 256),     # head_dim 64, ragged
    (32, 8, 128, 512, 256, 4096, 256),  # 32-row workgroups, as many as CUs
    (32, 8, 128, 640, 1024, 4096, 1024),  # 128-row workgroups, diagonal over many tiles
    (28, 4, 128, 300, 512, 4096, 512),  # 64-row workgroups, group of 7
])
def test_attention_outputs(hq, hkv, d, c, n, budget, chunk_max):
    """Eq. 1 alone: c + n <= budget in every case here, so nothing is scored or evicted and the
    block is appended.  Scores are checked where an eviction makes the library form them
    (test_scores_and_free_selection and every lock-step test)."""
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, budget, chunk_max, seed=c + n)
    assert err <= U.OUT_TOL, err
    k, v, idx, w, count, nxt = cache.decode_ready(0)
    assert count == c + n and nxt == c + n
    assert np.array_equal(idx[:, c:count].cpu().numpy(), np.broadcast_to(np.arange(c, c + n), (hkv, n)))
    cache.close()


@pytest.mark.parametrize("hq,hkv", [(46410, 1), (65900, 2)])
def test_many_query_heads_of_a_kv_head(hq, hkv):
    """A workgroup finds its KV head by a multiplication (csrc/divide.h): the last query heads of more than 46340 to a KV
    head, where query heads times their number per KV head pass 2^31."""
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, 64, 3, 5, 64, 16, seed=hq)
    assert err <= U.OUT_TOL, err
    cache.close()


@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("hq,hkv,d,c,n", [(8, 2, 128, 193, 300), (4, 4, 64, 70, 200), (4, 2, 128, 0, 129)])
def test_every_workgroup_shape(variant, hq, hkv, d, c, n):
    # the library picks the attention workgroup shape from the launch size; the tuning call forces the three shapes of
    # attention.hip in turn (the two that split the keys are picked by size: test_split_key_attention_edges)
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, 4096, 512, seed=7 * c + n + variant,
                                                    attention_shape=variant)
    assert err <= U.OUT_TOL, err
    cache.close()


@pytest.mark.parametrize("fused", [1, 0])
@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("hq,hkv,d,c,n,budget", [(8, 2, 128, 300, 200, 300), (4, 4, 64, 130, 190, 200), (6, 2, 128, 0, 129, 64)])
def test_every_workgroup_shape_scores(variant, fused, hq, hkv, d, c, n, budget):
    """Each workgroup shape of attention.hip, scoring inside the attention launch (its second sweep) or with the
    separate column-sum kernel reading the row statistics it leaves: scores and the selection made
    from them, with the shape forced."""
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, budget, 256, seed=11 + variant,
                                                    attention_shape=variant, fused=fused)
    assert err <= U.OUT_TOL, err
    scores_gpu, keep, dst = cache.debug_last(0)
    U.check_scores(scores_gpu.cpu().numpy(), scores_ref, n * (hq // hkv))
    cache.close()


@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("hq,hkv,d,c,n", [
    # tiles of 128 keys: one, two, three and more, odd and even numbers of plain ones; the cache ends with the first, the second or a later
    # tile, just before or behind its end; the block's rows end with a tile, one row behind it, one before
    (4, 2, 128, 0, 128), (4, 4, 64, 128, 128), (4, 2, 128, 128, 257), (4, 2, 128, 127, 129), (4, 4, 64, 129, 255), (4, 2, 128, 256, 128),
    (4, 2, 128, 255, 385), (4, 2, 64, 384, 256), (4, 2, 128, 385, 127), (2, 2, 128, 640, 384), (2, 1, 64, 1, 511), (2, 1, 128, 896, 129)])
def test_tiles_of_cache_and_block(variant, hq, hkv, d, c, n):
    """The loop over key tiles of attention.hip: whole ones through descriptors that move on, masked or not, and the others row by row."""
    budget = c + n - 1
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, budget, 512, seed=23 * c + n + variant, attention_shape=variant)
    assert err <= U.OUT_TOL, err
    U.check_scores(cache.debug_last(0)[0].cpu().numpy(), scores_ref, n * (hq // hkv))
    cache.close()


@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("hq,hkv,d,c,n", [
    # key blocks of 32: all of the cache, one that holds cached and new keys, a last one of one key, fewer than waves
    (4, 2, 128, 256, 160), (4, 2, 128, 255, 161), (4, 4, 64, 257, 128), (4, 2, 64, 33, 32), (4, 2, 128, 0, 33)])
def test_score_sweep_key_blocks(variant, hq, hkv, d, c, n):
    """The second sweep of attention.hip fetches a block of keys in whole rows, by one base address where the block lies in
    the cache or among the new keys entirely, row by row otherwise: scores at the edges of the two."""
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, max(c, n // 2), 192, seed=17 * c + n + variant,
                                                    attention_shape=variant)
    assert err <= U.OUT_TOL, err
    scores_gpu, keep, dst = cache.debug_last(0)
    U.check_scores(scores_gpu.cpu().numpy(), scores_ref, n * (hq // hkv))
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,c,n", [
    # keys split eight ways over 32-row tiles: fewer key blocks than waves, exactly as many, one more
    (4, 2, 128, 0, 1), (4, 4, 64, 0, 31), (4, 2, 128, 0, 32), (4, 4, 64, 1, 33), (4, 2, 128, 223, 32),
    (4, 2, 128, 224, 32), (4, 2, 64, 225, 64), (8, 2, 128, 31, 250), (6, 2, 64, 1025, 65),
    # four ways over 64-row tiles: a last tile of one row, of 32, of 33, nothing cached
    (28, 4, 128, 33, 321), (28, 4, 128, 300, 352), (16, 4, 64, 127, 545), (28, 4, 128, 0, 289)])
def test_split_key_attention_edges(hq, hkv, d, c, n):
    """Blocks too small to fill the chip, whose keys are split over the waves of a workgroup: outputs, and
    the scores that the same launch leaves when the block does not fit."""
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, max(c, n // 2, 1), 600, seed=31 * c + n)
    assert err <= U.OUT_TOL, err
    if c + n > max(c, n // 2, 1):                     # (one row of an empty cache fits and is not scored)
        scores_gpu, keep, dst = cache.debug_last(0)
        U.check_scores(scores_gpu.cpu().numpy(), scores_ref, n * (hq // hkv))
    cache.close()


@pytest.mark.parametrize("evicts", [False, True])
@pytest.mark.parametrize("hq,hkv,d,c,n", [
    # 32-row workgroups: a wave's blocks go on and on in the cache, then in the block's rows, with a part block at the end of either or of neither
    (4, 2, 128, 2048, 60), (4, 1, 128, 1100, 900), (4, 4, 64, 1025, 640), (8, 8, 64, 0, 1000), (16, 16, 128, 290, 500), (4, 2, 64, 4100, 33),
    # 64-row workgroups: the same with the tensors of two waves apart
    (28, 4, 128, 1500, 300), (32, 32, 128, 0, 700), (16, 4, 64, 1030, 600), (16, 16, 64, 95, 1200), (28, 28, 128, 1024, 320)])
def test_blocks_that_a_wave_moves_over(hq, hkv, d, c, n, evicts):
    """The split-key kernel's way from block to block: whole ones one after the other, and every change of kind, with scores and without."""
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, max(c, n // 2) if evicts else c + n, 1200, seed=7 * c + n)
    assert err <= U.OUT_TOL, err
    if evicts:
        U.check_scores(cache.debug_last(0)[0].cpu().numpy(), scores_ref, n * (hq // hkv))
    cache.close()


def _rows_of_a_workgroup(n, hq):
    """Query rows of the workgroups that csrc/plan.cpp picks for a block."""
    if -(-n // 128) * hq >= 192:
        return 128
    return 32 if -(-n // 32) * hq <= 256 else 64


KEPT_WEIGHTS = [
    # 32-row workgroups of eight waves: 1 to 8 key blocks per wave whose weights stay in registers (up to 6 at d 128),
    # and one more, for which the scores take a second sweep; one row past a tile, a last block of one key
    (4, 2, 128, 100, 33), (4, 2, 128, 481, 33), (4, 2, 128, 705, 32), (8, 2, 128, 930, 65), (4, 2, 128, 1216, 33),
    (4, 2, 128, 1472, 33), (4, 2, 128, 1473, 33), (4, 4, 64, 450, 33), (4, 2, 64, 704, 33), (4, 2, 64, 960, 64),
    (4, 2, 64, 1217, 1), (4, 2, 64, 1472, 33), (4, 2, 64, 1985, 33), (4, 2, 64, 1985, 65),
    # the fewest and the most blocks of a kernel: 9 and 16, 25 and 32; at d 64 8 and 9, 49 and 56, 57 and 64
    (4, 2, 128, 224, 33), (4, 2, 128, 448, 33), (4, 2, 128, 736, 33), (4, 2, 128, 960, 33), (4, 2, 64, 192, 33),
    (4, 2, 64, 224, 33), (4, 2, 64, 1504, 33), (4, 2, 64, 1728, 33), (4, 2, 64, 1760, 33), (4, 2, 64, 1984, 33)]


@pytest.mark.parametrize("scale", [0.0, 2.0])      # 2: logits of hundreds, so that references move in later blocks
@pytest.mark.parametrize("hq,hkv,d,c,n", KEPT_WEIGHTS)
def test_scores_from_kept_weights(hq, hkv, d, c, n, scale):
    """Scores out of the weights that a wave of the split-key kernel holds, for every number of blocks it is built for."""
    assert _rows_of_a_workgroup(n, hq) == 32
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, c, 96, seed=13 * c + n, scale=scale)
    assert err <= U.OUT_TOL, err
    scores_gpu, keep, dst = cache.debug_last(0)
    U.check_scores(scores_gpu.cpu().numpy(), scores_ref, n * (hq // hkv))
    cache.close()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_kept_weights_of_every_kernel(head_dim):
    """The cases above reach each kernel of this head dimension, with every number of blocks per wave that it serves."""
    with open(os.path.join(os.path.dirname(K.__file__), "csrc", "attention_split.hip")) as f:
        text = f.read()
    built = {int(x) for x in re.findall(r"if \(\(?e = prepare_shape<D, 1, (\d+)>", text)}
    built |= {int(x) for x in re.findall(r"if constexpr \(D == 64\) e = prepare_shape<D, 1, (\d+)>", text) if head_dim == 64}
    most = max(built)
    needed = {-(-(-(-c // 32) - (-n // 32)) // 8) for _, _, d, c, n in KEPT_WEIGHTS if d == head_dim}
    assert needed == set(range(1, most + 2))
    assert {min((k for k in built if k >= need), default=0) for need in needed} == built


@pytest.mark.parametrize("scale", [0.0, 2.0])
@pytest.mark.parametrize("hq,hkv,d,c,n", [
    # 64-row workgroups, whose first 16 key blocks stay in registers: 11, 15, 16 and 17 blocks for the latest rows; the last block
    # of 32-row workgroups (27 key blocks) and the first of 64-row ones (28); eight rounds of the second sweep (48)
    (28, 4, 128, 0, 330), (28, 4, 128, 100, 330), (28, 4, 128, 160, 330), (28, 4, 128, 161, 330), (16, 4, 64, 333, 512),
    (16, 4, 64, 333, 513), (28, 4, 128, 1024, 512)])
def test_scores_of_two_row_tiles(hq, hkv, d, c, n, scale):
    """Scores of the split-key kernel with two row tiles: out of kept weights of both tiles, and a second sweep for the rest."""
    assert _rows_of_a_workgroup(n, hq) == (32 if (hq, n) == (16, 512) else 64)
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, max(c, 1), max(512, n), seed=19 * c + n, scale=scale)
    assert err <= U.OUT_TOL, err
    scores_gpu, keep, dst = cache.debug_last(0)
    U.check_scores(scores_gpu.cpu().numpy(), scores_ref, n * (hq // hkv))
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,c,n", [
    # 32-row workgroups: waves with no block, one, two; the cache's part block first, in between, last of a wave
    (4, 4, 64, 0, 5), (4, 2, 128, 1, 30), (4, 2, 64, 257, 33), (6, 2, 128, 290, 63), (4, 4, 64, 511, 1),
    # 64-row workgroups: the part block of the cache in every wave; one, two and three rounds; an odd and an even number of them
    (28, 4, 128, 0, 293), (28, 4, 128, 31, 300), (28, 4, 128, 33, 300), (32, 32, 128, 65, 290), (16, 4, 64, 97, 530), (28, 4, 64, 129, 330)])
def test_rows_past_the_end_of_a_block(hq, hkv, d, c, n):
    """Key blocks of the split-key kernel that end early: what lies behind the cached entries and behind the block's rows in memory is
    NaN and stays out of outputs and scores."""
    _rows_past_the_end(hq, hkv, d, c, n)


@pytest.mark.parametrize("shape", [0, 1, 2])
@pytest.mark.parametrize("hq,hkv,d,c,n", [
    # tiles of 128 keys: the first holds all there is, or cached and new keys; a later one does; whole tiles and a last one of a few keys
    (4, 4, 64, 0, 5), (4, 2, 128, 127, 129), (4, 4, 64, 129, 255), (4, 2, 128, 300, 200), (4, 2, 64, 512, 130), (2, 1, 128, 900, 641)])
def test_rows_past_the_end_of_a_tile(shape, hq, hkv, d, c, n):
    """The same for the key tiles of the shapes that a caller can force."""
    _rows_past_the_end(hq, hkv, d, c, n, shape)


def _rows_past_the_end(hq, hkv, d, c, n, shape=-1):
    rng = np.random.default_rng(100 * c + n)
    cache = K.Cache(1, hq, hkv, d, c + n - 1, n, [Segment(0, 100000, 0)], device=DEV)
    cache.set_attention_shape(shape)
    k_all, v_all, q = _rand_bits(rng, (c + n, hkv, d)), _rand_bits(rng, (c + n, hkv, d)), _rand_bits(rng, (n, hq, d))
    oc = O.LayerCache(hkv, d, c + n - 1)
    if c:
        oc.compact(0, *(O.bf16_bits_to_f64(x[:c]) for x in (k_all, v_all)), np.zeros((hkv, c), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    for t in cache.decode_ready(0)[:2]:
        t[:, c:] = float("nan")
    cache.set_state(0, c, c)
    fresh = []
    for x in (k_all, v_all):
        wide = torch.full((n + 40, hkv, d), float("nan"), dtype=torch.bfloat16, device=DEV)
        wide[:n] = U.bits_to_torch(x[c:])
        fresh.append(wide[:n])
    out = cache.prefill_chunk(0, c, U.bits_to_torch(q), *fresh)
    out_ref, scores_ref = oc.attend(c, O.bf16_bits_to_f64(q), O.bf16_bits_to_f64(k_all[c:]), O.bf16_bits_to_f64(v_all[c:]), None)
    err = U.out_rel_err(U.torch_bf16_to_f64(out), out_ref)
    assert err <= U.OUT_TOL, err
    cache.compact(0)
    U.check_scores(cache.debug_last(0)[0].cpu().numpy(), scores_ref, n * (hq // hkv))
    cache.close()


@pytest.mark.parametrize("fused", [1, 0])
@pytest.mark.parametrize("hq,hkv,d,c,n,budget,chunk_max,scale", [
    (4, 4, 64, 128, 64, 128, 64, 0.0),
    (8, 2, 128, 200, 150, 200, 256, 0.0),
    (32, 8, 128, 512, 300, 512, 512, 0.0),
    (28, 4, 128, 1024, 512, 1024, 512, 0.0),
    (4, 2, 128, 96, 40, 100, 64, 0.25),     # explicit scale, cache below budget going over it
    (32, 8, 128, 2048, 1024, 2048, 1024, 0.0),   # the bench shape at steady state
    (2, 2, 64, 6144, 2048, 6144, 2048, 0.0),     # the candidate limit: 8192 per head
    (4, 1, 64, 37, 5, 40, 8, 0.0),               # a handful of rows, one KV head
    (16, 1, 64, 100, 520, 256, 520, 0.0),        # 16 heads per KV head x 9 row tiles: past the fused limit
])
def test_scores_and_free_selection(hq, hkv, d, c, n, budget, chunk_max, scale, fused):
    """The library's own scores (out of the attention launch's second sweep, or from the separate
    column-sum kernel), and the selection it makes from them."""
    cache, oc, err, scores_ref, (q64, k64, v64) = _attention_case(hq, hkv, d, c, n, budget, chunk_max,
                                                                  seed=7 * c + n, scale=scale, fused=fused)
    assert err <= U.OUT_TOL, err
    scores_gpu, keep, dst = cache.debug_last(0)
    scores_gpu = scores_gpu.cpu().numpy()
    g = hq // hkv
    U.check_scores(scores_gpu, scores_ref, n * g)
    np.testing.assert_allclose(scores_gpu.sum(axis=1), n * g, rtol=1e-4)      # softmax rows sum to 1
    # selection on the GPU's own fp32 scores must be what the definition gives for those scores
    tok = np.concatenate([oc.idx, np.broadcast_to(np.arange(c, c + n), (hkv, n))], axis=1)
    keep = keep.cpu().numpy().astype(bool)
    for hk in range(hkv):
        want = O.select_keep(scores_gpu[hk], tok[hk], budget)
        assert np.array_equal(keep[hk], want)
    k, v, idx, w, count, nxt = cache.decode_ready(0)
    assert count == budget and nxt == c + n
    idx = idx.cpu().numpy()
    for hk in range(hkv):
        assert sorted(idx[hk].tolist()) == sorted(tok[hk][keep[hk]].tolist())
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,c,n,budget,chunk_max,n_obs,scale", [
    (4, 4, 64, 128, 64, 128, 64, 16, 0.0),
    (8, 2, 128, 200, 150, 200, 256, 33, 0.0),         # ragged proxy rows
    (4, 2, 128, 96, 40, 100, 64, 1, 0.25),            # a single proxy query, explicit scale
    (28, 4, 128, 1024, 512, 1024, 512, 512, 0.0),     # as many proxy queries as a block holds
    (32, 8, 128, 2048, 1024, 2048, 1024, 64, 0.0),    # the bench shape with a 64-token prompt
    (2, 2, 64, 6144, 2048, 6144, 2048, 100, 0.0),     # the candidate limit
    (4, 2, 64, 0, 96, 32, 96, 8, 0.0),                # empty cache, block larger than the budget
    # enough (query head, row tile) items per KV head for the row-statistics kernel to give a
    # workgroup several of them: 32 items in equal shares; 21 items, the last share is a single one
    (16, 2, 64, 6144, 2048, 6144, 2048, 100, 0.0),
    (28, 4, 64, 6144, 2048, 6144, 2048, 70, 0.0),
])
def test_proxy_query_scores_and_selection(hq, hkv, d, c, n, budget, chunk_max, n_obs, scale):
    """Scores taken with proxy queries (every candidate visible to each of them), the attention
    output unchanged, and the selection made from those scores."""
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, budget, chunk_max, seed=3 * c + n + n_obs,
                                                    scale=scale, n_obs=n_obs)
    assert err <= U.OUT_TOL, err
    scores_gpu, keep, dst = cache.debug_last(0)
    scores_gpu = scores_gpu.cpu().numpy()
    g = hq // hkv
    U.check_scores(scores_gpu, scores_ref, n_obs * g)
    np.testing.assert_allclose(scores_gpu.sum(axis=1), n_obs * g, rtol=1e-4)
    tok = np.concatenate([oc.idx, np.broadcast_to(np.arange(c, c + n), (hkv, n))], axis=1)
    keep = keep.cpu().numpy().astype(bool)
    for hk in range(hkv):
        assert np.array_equal(keep[hk], O.select_keep(scores_gpu[hk], tok[hk], budget))
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,c,n,budget,chunk_max", [
    (4, 4, 64, 128, 64, 128, 64),
    (8, 2, 128, 200, 150, 200, 256),
    (32, 8, 128, 2048, 1024, 2048, 1024),     # the bench shape
    (2, 2, 64, 6144, 2048, 6144, 2048),       # the candidate limit
    (4, 2, 64, 0, 96, 32, 96),                # empty cache, block larger than the budget
    (4, 1, 128, 37, 5, 40, 8),
])
def test_keydiff_scores_and_selection(hq, hkv, d, c, n, budget, chunk_max):
    """Query-agnostic scores (minus the cosine to the mean candidate key), the attention output
    unchanged, and the selection made from those scores."""
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, budget, chunk_max, seed=5 * c + n, keydiff=True)
    assert err <= U.OUT_TOL, err
    scores_gpu, keep, dst = cache.debug_last(0)
    scores_gpu = scores_gpu.cpu().numpy()
    # fp32 sums of at most 8192 terms against float64: a cosine is off by a few 1e-6 at most
    assert np.abs(scores_gpu - scores_ref).max() <= 2e-5
    tok = np.concatenate([oc.idx, np.broadcast_to(np.arange(c, c + n), (hkv, n))], axis=1)
    keep = keep.cpu().numpy().astype(bool)
    for hk in range(hkv):
        assert np.array_equal(keep[hk], O.select_keep(scores_gpu[hk], tok[hk], budget))
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,c,n", [(4, 2, 64, 100, 150), (8, 2, 128, 256, 300), (4, 4, 128, 0, 96),
                                          (8, 2, 128, 1280, 300),    # the runaway shows up in tiles that no longer track maxima
                                          (32, 8, 128, 1536, 1024)])  # ... and in the eight-wave shape
def test_runaway_logits_take_the_careful_path(hq, hkv, d, c, n):
    """Logits that climb by hundreds of nats along the keys: the fixed softmax reference of the
    fast loop would overflow, so the kernel must detect it and redo the rows exactly."""
    from kvp_workload import f32_to_bf16_bits
    rng = np.random.default_rng(d + c)
    budget, chunk_max = 4096, max(512, n)
    segs = [Segment(0, 100000, 0)]
    cache = K.Cache(1, hq, hkv, d, budget, chunk_max, segs, merge=False, device=DEV)
    tot = c + n
    ramp = (np.arange(tot, dtype=np.float32) / tot)[:, None, None]                   # later keys score higher
    k_all = (8.0 * ramp * np.ones((tot, hkv, d), dtype=np.float32)) + 0.05 * rng.standard_normal((tot, hkv, d)).astype(np.float32)
    v_all = rng.standard_normal((tot, hkv, d)).astype(np.float32)
    q = (8.0 * np.ones((n, hq, d), dtype=np.float32)) + 0.05 * rng.standard_normal((n, hq, d)).astype(np.float32)
    kb, vb, qb = f32_to_bf16_bits(k_all), f32_to_bf16_bits(v_all), f32_to_bf16_bits(q)
    oc = O.LayerCache(hkv, d, budget)
    if c:
        oc.compact(0, O.bf16_bits_to_f64(kb[:c]), O.bf16_bits_to_f64(vb[:c]), np.zeros((hkv, c), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, c)
    out = cache.prefill_chunk(0, c, U.bits_to_torch(qb), U.bits_to_torch(kb[c:]), U.bits_to_torch(vb[c:]))
    out_ref, scores_ref = oc.attend(c, O.bf16_bits_to_f64(qb), O.bf16_bits_to_f64(kb[c:]), O.bf16_bits_to_f64(vb[c:]))
    assert np.isfinite(U.torch_bf16_to_f64(out)).all()
    assert U.out_rel_err(U.torch_bf16_to_f64(out), out_ref) <= U.OUT_TOL
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,c,n", [
    (4, 2, 128, 700, 150), (16, 4, 64, 1111, 333),       # 32-row workgroups, the keys split eight ways
    (28, 4, 128, 0, 352), (28, 4, 128, 1025, 321), (16, 4, 64, 700, 545),      # 64-row workgroups, four ways
    (32, 8, 128, 1536, 1024)])                           # 128-row workgroups
def test_scores_after_runaway_logits(hq, hkv, d, c, n):
    """Logits that climb by hundreds of nats along the keys, in a block that evicts: a row's softmax reference moves in
    every key block of a wave, and the scores come from the normalisers that this leaves."""
    from kvp_workload import f32_to_bf16_bits
    rng = np.random.default_rng(d + c + n)
    budget = max(c, n // 2)
    cache = K.Cache(1, hq, hkv, d, budget, n, [Segment(0, 100000, 0)], merge=False, device=DEV)
    tot = c + n
    # raw products up to 32 d: fp32 sums of them are off by 8 half units in the last place at most, 2e-4 nats
    ramp = 8.0 * np.arange(tot, dtype=np.float32)[:, None, None] / tot
    kb = f32_to_bf16_bits(ramp + 0.05 * rng.standard_normal((tot, hkv, d)).astype(np.float32))
    vb = _rand_bits(rng, (tot, hkv, d))
    qb = f32_to_bf16_bits(4.0 + 0.05 * rng.standard_normal((n, hq, d)).astype(np.float32))
    q64, k64, v64 = (O.bf16_bits_to_f64(x) for x in (qb, kb, vb))
    oc = O.LayerCache(hkv, d, budget)
    if c:
        oc.compact(0, k64[:c], v64[:c], np.zeros((hkv, c), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, c)
    out_ref, scores_ref = oc.attend(c, q64, k64[c:], v64[c:])
    out = cache.prefill_chunk(0, c, U.bits_to_torch(qb), U.bits_to_torch(kb[c:]), U.bits_to_torch(vb[c:]))
    cache.compact(0)
    assert U.out_rel_err(U.torch_bf16_to_f64(out), out_ref) <= U.OUT_TOL
    scores, kept, _ = (x.cpu().numpy() for x in cache.debug_last(0))
    U.check_scores(scores, scores_ref, n * (hq // hkv))
    tok = np.concatenate([oc.idx, np.broadcast_to(np.arange(c, tot), (hkv, n))], axis=1)
    for hk in range(hkv):
        assert np.array_equal(kept[hk].astype(bool), O.select_keep(scores[hk], tok[hk], budget))
    cache.close()


@pytest.mark.parametrize("scale", [0.0, 1e-38])         # 1e-38: the margin for a row's reference, in units of the dot product, is infinite
@pytest.mark.parametrize("hq,hkv,d,c,n", [(4, 2, 64, 512, 33), (4, 2, 128, 515, 70), (28, 4, 128, 520, 300), (16, 4, 64, 517, 530)])
def test_first_keys_at_minus_infinity(hq, hkv, d, c, n, scale):
    """Split-key kernel: the first 256 keys have logits of minus infinity in every other row and of plus infinity in the
    rows between them.  The former average over the other keys; the latter are not finite."""
    assert _rows_of_a_workgroup(n, hq) < 128
    rng = np.random.default_rng(c + n)
    cache = K.Cache(1, hq, hkv, d, c + n, n, [Segment(0, 100000, 0)], softmax_scale=scale, device=DEV)
    k_all, v_all, q = _rand_bits(rng, (c + n, hkv, d)), _rand_bits(rng, (c + n, hkv, d)), _rand_bits(rng, (n, hq, d))
    q[0::2, :, 5] &= 0x7FFF
    q[1::2, :, 5] |= 0x8000
    k_all[:256, :, 5] = 0xFF80
    k64, v64, q64 = (O.bf16_bits_to_f64(x) for x in (k_all, v_all, q))
    oc = O.LayerCache(hkv, d, c + n)
    oc.compact(0, k64[:c], v64[:c], np.zeros((hkv, c), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, c)
    out = cache.prefill_chunk(0, c, U.bits_to_torch(q), U.bits_to_torch(k_all[c:]), U.bits_to_torch(v_all[c:]))
    finite = O.LayerCache(hkv, d, c + n)
    finite.compact(0, k64[256:c], v64[256:c], np.zeros((hkv, c - 256), dtype=np.float32))
    out_ref, _ = finite.attend(c - 256, q64, k64[c:], v64[c:], scale or None)
    err = U.out_rel_err(U.torch_bf16_to_f64(out)[0::2], out_ref[0::2])
    assert err <= U.OUT_TOL, err
    cache.close()


@pytest.mark.parametrize("value", ["nan", "inf", "huge"])     # huge: finite, but logits up to infinity
@pytest.mark.parametrize("hq,hkv,d,c,n,fused", [
    (4, 2, 128, 100, 33, 1), (4, 2, 128, 1216, 65, 1), (4, 4, 64, 450, 60, 1), (4, 2, 64, 1985, 65, 1),    # 32-row workgroups
    (28, 4, 128, 0, 330, 1), (28, 4, 128, 161, 330, 1), (16, 4, 64, 333, 545, 1),                          # 64-row workgroups
    (32, 8, 128, 256, 800, 1),                                                                             # 128-row workgroups
    (8, 2, 128, 130, 150, 0)])                                                                             # separate kernel
def test_scores_beside_a_row_that_is_not_finite(hq, hkv, d, c, n, fused, value):
    """Rows whose logits are not finite spoil the scores of the keys that they see, and of no others: the block's later keys,
    in the same block of 32 among them, score what the other rows give them."""
    rng = np.random.default_rng(23 * c + n)
    cache = K.Cache(1, hq, hkv, d, max(c, 1), n, [Segment(0, 100000, 0)], merge=False, device=DEV)
    cache.set_score_sweep(fused)
    qb, kb, vb = _rand_bits(rng, (n, hq, d)), _rand_bits(rng, (c + n, hkv, d)), _rand_bits(rng, (c + n, hkv, d))
    q64, k64, v64 = (O.bf16_bits_to_f64(x) for x in (qb, kb, vb))
    group = hq // hkv
    bad = {0: 3, hkv - 1: n // 2 + 1}                 # KV head -> row; the last of its query heads
    qt = U.bits_to_torch(qb)
    for hk, row in bad.items():
        q64[row, hk * group + group - 1] = 0.0        # a row that says nothing about later keys, either
        qt[row, hk * group + group - 1, 5] = {"nan": float("nan"), "inf": float("inf"), "huge": 3e38}[value]
    oc = O.LayerCache(hkv, d, max(c, 1))
    if c:
        oc.compact(0, k64[:c], v64[:c], np.zeros((hkv, c), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, c)
    out_ref, scores_ref = oc.attend(c, q64, k64[c:], v64[c:])
    out = cache.prefill_chunk(0, c, qt, U.bits_to_torch(kb[c:]), U.bits_to_torch(vb[c:]))
    cache.compact(0)
    scores = cache.debug_last(0)[0].cpu().numpy()
    good = np.ones((n, hq), dtype=bool)
    seen = np.zeros((hkv, c + n), dtype=bool)
    for hk, row in bad.items():
        good[row, hk * group + group - 1] = False
        seen[hk, :c + row + 1] = True
    assert U.out_rel_err(U.torch_bf16_to_f64(out)[good], out_ref[good]) <= U.OUT_TOL
    U.check_scores(scores[~seen], scores_ref[~seen], n * group)
    if value != "huge":
        assert not np.isfinite(scores[seen]).any()
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,c,n_tail,budget,chunk_max,scale", [
    (4, 4, 64, 0, 1, 256, 64, 0.0),          # nothing cached: the current token alone
    (4, 2, 128, 63, 1, 256, 64, 0.0),        # exactly one 64-key group
    (8, 2, 128, 193, 7, 256, 64, 0.0),       # ragged groups, a short tail
    (4, 4, 64, 300, 70, 512, 128, 0.25),     # the tail spans a group boundary; explicit scale
    (32, 8, 128, 2048, 1, 2048, 1024, 0.0),  # the bench shape
    (32, 8, 128, 2048, 513, 2048, 1024, 0.0),
    (28, 4, 128, 1024, 33, 1024, 512, 0.0),  # seven query heads per KV head
    (16, 1, 64, 100, 3, 128, 16, 0.0),       # sixteen per KV head, little scratch
    (2, 2, 64, 6144, 5000, 6144, 2048, 0.0),  # many groups per wave
])
def test_decode_step(hq, hkv, d, c, n_tail, budget, chunk_max, scale):
    """One generation step over a preloaded cache and a tail of generated tokens."""
    rng = np.random.default_rng(1000 + c + n_tail)
    cache = K.Cache(1, hq, hkv, d, budget, chunk_max, [Segment(0, 100000, 0)], merge=False, softmax_scale=scale, device=DEV)
    oc = O.LayerCache(hkv, d, budget)
    if c:
        kb0, vb0 = _rand_bits(rng, (c, hkv, d)), _rand_bits(rng, (c, hkv, d))
        oc.compact(0, O.bf16_bits_to_f64(kb0), O.bf16_bits_to_f64(vb0), np.zeros((hkv, c), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, c)
    qb, kb, vb = _rand_bits(rng, (hq, d), 2.0), _rand_bits(rng, (n_tail, hkv, d)), _rand_bits(rng, (n_tail, hkv, d))
    q64, k64, v64 = (O.bf16_bits_to_f64(x) for x in (qb, kb, vb))
    _, _, k_all, v_all = oc.candidates(c, k64, v64)
    ref = O.decode_step(q64, k_all, v_all, scale or None)
    out = cache.decode_step(0, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
    err = U.out_rel_err(U.torch_bf16_to_f64(out), ref)
    assert err <= U.OUT_TOL, err
    # the cache is untouched: the same call again gives the same bits, and so does the
    # block entry point for a one-row block when the tail is the current token alone
    again = cache.decode_step(0, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
    assert torch.equal(out, again)
    if n_tail == 1 and c < budget:
        blk = cache.prefill_chunk(0, c, U.bits_to_torch(qb)[None], U.bits_to_torch(kb), U.bits_to_torch(vb))
        assert U.out_rel_err(U.torch_bf16_to_f64(blk[0]), ref) <= U.OUT_TOL
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,n_keys", [
    # one workgroup per query head: edges of its rows per thread, and the first keys beyond
    (8, 2, 128, 64), (8, 2, 128, 65), (8, 2, 128, 255), (8, 2, 128, 257), (7, 7, 128, 640), (7, 1, 128, 641), (4, 4, 64, 513), (12, 4, 64, 1280), (12, 4, 64, 1281),
    # partial results: a workgroup whose last waves have no key, more than 48 partials to fold
    (10, 1, 128, 705), (4, 4, 64, 64 * 49 + 1)])
def test_decode_step_edges(hq, hkv, d, n_keys):
    rng = np.random.default_rng(n_keys)
    c = n_keys - 5
    cache = K.Cache(1, hq, hkv, d, c, 64, [Segment(0, 100000, 0)], device=DEV)
    oc = O.LayerCache(hkv, d, c)
    kb0, vb0 = _rand_bits(rng, (c, hkv, d)), _rand_bits(rng, (c, hkv, d))
    oc.compact(0, O.bf16_bits_to_f64(kb0), O.bf16_bits_to_f64(vb0), np.zeros((hkv, c), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, c)
    qb, kb, vb = _rand_bits(rng, (hq, d), 2.0), _rand_bits(rng, (5, hkv, d)), _rand_bits(rng, (5, hkv, d))
    _, _, k_all, v_all = oc.candidates(c, O.bf16_bits_to_f64(kb), O.bf16_bits_to_f64(vb))
    ref = O.decode_step(O.bf16_bits_to_f64(qb), k_all, v_all)
    out = cache.decode_step(0, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
    assert U.out_rel_err(U.torch_bf16_to_f64(out), ref) <= 5e-3      # fp32 throughout: the rounding of the output to bf16 alone
    cache.close()


@pytest.mark.parametrize("d,n_keys", [(64, 64 * 21 + 1), (128, 64 * 11 + 1), (128, 64 * 11 - 1)])
@pytest.mark.parametrize("hq,hkv", [(3, 1), (8, 2), (5, 1), (12, 2), (7, 1), (16, 2), (9, 1)])
def test_decode_step_of_every_group(hq, hkv, d, n_keys):
    """More keys than one workgroup takes, for the numbers of query heads per KV head that the kernel is built for, and others."""
    test_decode_step_edges(hq, hkv, d, n_keys)


@pytest.mark.parametrize("d,c", [(64, 90), (128, 90), (128, 900)])       # the kernel of few keys, and of many
@pytest.mark.parametrize("keys,queries", [(0, 0), (-128, 125), (125, -128)])
def test_decode_logits(d, c, keys, queries):
    """Logits of a decode step to fp32 rounding: keys that differ by little, under a large softmax scale.  Keys or queries times
    2^-128 are denormal numbers, the others large."""
    rng = np.random.default_rng(d + c)
    hq, hkv = 8, 4
    scale = 32.0 * 2.0 ** -(keys + queries)
    base = np.round(np.clip(rng.standard_normal((1, hkv, d)), -3, 3) * 32) / 32
    rows = np.repeat(base, c + 5, axis=0)                  # one channel of each is off by up to 3/32: bf16 has these numbers
    rows[np.arange(c + 5)[:, None], np.arange(hkv)[None], rng.integers(0, d, (c + 5, hkv))] += rng.integers(0, 4, (c + 5, hkv)) / 32
    q = np.round(np.clip(rng.standard_normal((hq, d)), -3, 3) * 32) / 32
    kb, qb = O.f64_to_bf16_bits(rows * 2.0 ** keys), O.f64_to_bf16_bits(q * 2.0 ** queries)
    vb = _rand_bits(rng, (c + 5, hkv, d))
    q64, k64, v64 = (O.bf16_bits_to_f64(x) for x in (qb, kb, vb))
    cache = K.Cache(1, hq, hkv, d, c, 64, [Segment(0, 100000, 0)], merge=False, softmax_scale=scale, device=DEV)
    oc = O.LayerCache(hkv, d, c)
    oc.compact(0, k64[:c], v64[:c], np.zeros((hkv, c), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, c)
    _, _, k_all, v_all = oc.candidates(c, k64[c:], v64[c:])
    ref = O.decode_step(q64, k_all, v_all, scale)
    out = U.torch_bf16_to_f64(cache.decode_step(0, U.bits_to_torch(qb), U.bits_to_torch(kb[c:]), U.bits_to_torch(vb[c:])))
    # a logit is the sum of d products, each of which meets at most twelve roundings (8 of a lane, sixteen lanes); an error e of the
    # logits changes a weight by a factor of exp(2 e) at most; the output is rounded to bf16 once
    most = np.abs(q64).sum(axis=1).max() * np.abs(k64).max()
    e = scale * 12 * 2.0 ** -24 * most
    assert e < 0.02
    assert np.abs(out - ref).max() <= (2.1 * e + 2.0 ** -8) * np.abs(v64).max()
    cache.close()


ONE_WORKGROUP = [(8, 2, 128, 100), (4, 4, 128, 333), (8, 2, 128, 560), (8, 2, 64, 900)]      # per query head, few rows per thread and many


@pytest.mark.parametrize("hq,hkv,d,n_keys", ONE_WORKGROUP + [
    (4, 4, 128, 900), (4, 2, 128, 900), (8, 2, 64, 1500),                        # partial results, by vector instructions
    (6, 2, 128, 900), (8, 2, 128, 8900), (14, 2, 128, 8900), (20, 2, 128, 8900), (32, 2, 128, 700)])      # by matrix instructions, and several tiles
@pytest.mark.parametrize("kind", ["growing", "denormal", "infinite"])
def test_decode_values(hq, hkv, d, n_keys, kind):
    """Weights against references that later keys leave behind, values too small for a normal number, and infinite ones."""
    _decode_values(hq, hkv, d, n_keys, kind)


@pytest.mark.parametrize("hq,hkv,d,n_keys", ONE_WORKGROUP)
def test_decode_values_near_the_largest(hq, hkv, d, n_keys):
    """Sums that only the small weights of their values keep finite, over keys that some waves have to themselves."""
    _decode_values(hq, hkv, d, n_keys, "large")


def _decode_values(hq, hkv, d, n_keys, kind):
    rng = np.random.default_rng(n_keys + hq)
    tail = 2900 if n_keys > 6000 else 50
    c, g = n_keys - tail, hq // hkv
    kb, vb, qb = _rand_bits(rng, (n_keys, hkv, d)), _rand_bits(rng, (n_keys, hkv, d)), _rand_bits(rng, (hq, d))
    k64, v64, q64 = O.bf16_bits_to_f64(kb), O.bf16_bits_to_f64(vb), O.bf16_bits_to_f64(qb)
    if kind == "growing":
        k64 = O.bf16_bits_to_f64(f32_to_bf16_bits((k64 * np.linspace(0.1, 4, n_keys)[:, None, None]).astype(np.float32)))
        k64[rng.permutation(n_keys)[:n_keys // 3]] = 0.0
    elif kind == "denormal":
        v64 = O.bf16_bits_to_f64(f32_to_bf16_bits((v64 * 2.0 ** -128).astype(np.float32)))
    elif kind == "large":
        q64[:] = rng.choice([-1.0, 1.0], size=d)
        large = np.arange(n_keys) % 64 // 8 == 2
        k64[large] = -2 * q64[0]             # 2 sqrt(d) below the mean of the others' logits
        v64[large] = 2.0 ** 127
    else:
        v64[rng.integers(n_keys // 2), 0, 3] = np.inf
        v64[n_keys // 3, 0, 5] = -np.inf     # (not among the last keys, whose values and results are read again for what is not there)
        v64[[0, n_keys // 2], 0, 7] = np.inf, -np.inf
    to_gpu = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.bfloat16).to(DEV)      # (exact)
    cache = K.Cache(1, hq, hkv, d, c, min(c, 512), [Segment(0, 100000, 0)], merge=False, device=DEV)
    k, v, token, weight, _, _ = cache.decode_ready(0)
    k.copy_(to_gpu(k64[:c].transpose(1, 0, 2)))
    v.copy_(to_gpu(v64[:c].transpose(1, 0, 2)))
    token.copy_(torch.arange(c, device=DEV, dtype=torch.int32).expand(hkv, c))
    weight.fill_(1.0)
    cache.set_state(0, c, c)
    out = U.torch_bf16_to_f64(cache.decode_step(0, to_gpu(q64), to_gpu(k64[c:]), to_gpu(v64[c:])))
    with np.errstate(invalid="ignore"):
        ref = O.decode_step(q64, k64.transpose(1, 0, 2), v64.transpose(1, 0, 2))
    if kind == "infinite":
        assert np.isposinf(ref[:g, 3]).all() and np.isneginf(ref[:g, 5]).all() and np.isnan(ref[:g, 7]).all()
        assert np.array_equal(np.isposinf(out), np.isposinf(ref)) and np.array_equal(np.isneginf(out), np.isneginf(ref))
        assert np.array_equal(np.isnan(out), np.isnan(ref))
        ok = np.isfinite(ref)
        assert np.abs(out[ok] - ref[ok]).max() <= 5e-3 * np.abs(ref[ok]).max()
    elif kind == "denormal":     # half a unit of the smallest bf16 numbers, and as much for the fp32 sums of two roundings
        assert np.abs(out - ref).max() <= 2.0 ** -133 + 5e-3 * np.abs(ref).max()
    else:
        assert U.out_rel_err(out, ref) <= 5e-3       # fp32 throughout: the rounding of the output to bf16 alone
    cache.close()


@pytest.mark.parametrize("hkv", [8192, 8193, 65537])       # one launch of few keys, two of more KV heads than 32-bit offsets reach
def test_decode_step_of_many_kv_heads(hkv):
    rng = np.random.default_rng(hkv)
    cache = K.Cache(1, hkv, hkv, 64, 3, 1, [Segment(0, 100, 0)], merge=False, device=DEV)
    oc = O.LayerCache(hkv, 64, 3)
    kb0, vb0, kb, vb = (_rand_bits(rng, (m, hkv, 64)) for m in (3, 3, 2, 2))
    oc.compact(0, O.bf16_bits_to_f64(kb0), O.bf16_bits_to_f64(vb0), np.zeros((hkv, 3), dtype=np.float32))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, 3, 3)
    qb = _rand_bits(rng, (hkv, 64))
    _, _, k_all, v_all = oc.candidates(3, O.bf16_bits_to_f64(kb), O.bf16_bits_to_f64(vb))
    ref = O.decode_step(O.bf16_bits_to_f64(qb), k_all, v_all)
    out = cache.decode_step(0, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
    assert U.out_rel_err(U.torch_bf16_to_f64(out), ref) <= 5e-3      # as above
    cache.close()


def test_decode_step_after_prefill():
    """Prefill a layer block by block, then generate three tokens over what it kept."""
    wl = get_workload("tiled_image")
    cache = K.Cache(1, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk, wl.segments, merge=True, device=DEV)
    qb, kb, vb = layer_inputs(wl, 0)
    oc = U.lockstep_layer(wl, 0, cache, qb, kb, vb, True, own_scores=False)
    rng = np.random.default_rng(5)
    hq, hkv, d = wl.n_q_heads, wl.n_kv_heads, wl.head_dim
    kt, vt = _rand_bits(rng, (3, hkv, d)), _rand_bits(rng, (3, hkv, d))
    for step in range(1, 4):
        qb = _rand_bits(rng, (hq, d), 2.0)
        _, _, k_all, v_all = oc.candidates(wl.n_tokens, O.bf16_bits_to_f64(kt[:step]), O.bf16_bits_to_f64(vt[:step]))
        ref = O.decode_step(O.bf16_bits_to_f64(qb), k_all, v_all)
        out = cache.decode_step(0, U.bits_to_torch(qb), U.bits_to_torch(kt[:step]), U.bits_to_torch(vt[:step]))
        assert U.out_rel_err(U.torch_bf16_to_f64(out), ref) <= U.OUT_TOL
    cache.close()


def test_select_ties_and_override():
    """All scores equal: the lowest token indices stay (ties to the lower index)."""
    hq = hkv = 2
    d, c, n, budget = 64, 96, 64, 96
    rng = np.random.default_rng(5)
    segs = [Segment(0, 100000, 0)]
    cache = K.Cache(1, hq, hkv, d, budget, 64, segs, merge=False, device=DEV)
    oc = O.LayerCache(hkv, d, budget)
    kb0 = _rand_bits(rng, (c, hkv, d))
    oc.compact(0, O.bf16_bits_to_f64(kb0), O.bf16_bits_to_f64(kb0), np.zeros((hkv, c), dtype=np.float32))
    perm = np.stack([rng.permutation(c) for _ in range(hkv)])
    oc.idx = np.take_along_axis(oc.idx, perm, axis=1)
    oc.K = np.take_along_axis(oc.K, perm[:, :, None], axis=1)
    oc.V = np.take_along_axis(oc.V, perm[:, :, None], axis=1)
    qb, kb, vb = _rand_bits(rng, (n, hq, d)), _rand_bits(rng, (n, hkv, d)), _rand_bits(rng, (n, hkv, d))
    for pattern in ("equal", "two_levels", "negative"):
        sc = np.zeros((hkv, c + n), dtype=np.float32)
        if pattern == "two_levels":
            sc[:, ::3] = 1.5
        if pattern == "negative":
            sc = -np.abs(rng.standard_normal((hkv, c + n))).astype(np.float32)
            sc[:, 5] = -0.0
        oc2 = O.LayerCache(hkv, d, budget)
        oc2.idx, oc2.w, oc2.K, oc2.V, oc2.count = oc.idx.copy(), oc.w.copy(), oc.K.copy(), oc.V.copy(), c
        U.upload_state(cache, 0, oc2)
        cache.set_state(0, c, c)
        cache.prefill_chunk(0, c, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
        cache.compact(0, torch.from_numpy(sc).to(DEV))
        rec = oc2.compact(c, O.bf16_bits_to_f64(kb), O.bf16_bits_to_f64(vb), sc)
        _, keep, _ = cache.debug_last(0)
        assert np.array_equal(keep.cpu().numpy().astype(bool), rec["keep"]), pattern
        U.compare_state(cache, 0, oc2)
        if pattern == "equal":
            _, _, idx, _, _, _ = cache.decode_ready(0)
            assert sorted(idx[0].cpu().numpy().tolist()) == list(range(budget))
    cache.close()


def _layer_cases():
    """Every layer of every workload, merge on; plus the paper's own method (merge off) on a few."""
    cases = []
    for name in ("tiny", "single_image", "tiled_image", "video", "long_video"):
        wl = get_workload(name)
        cases += [(name, True, layer) for layer in range(wl.n_layers)]
    cases += [("tiny", False, 0), ("single_image", False, 2), ("tiled_image", False, 1), ("video", False, 9),
              ("long_video", False, 17)]
    return cases


@pytest.mark.parametrize("name,merge,layer", _layer_cases())
def test_lockstep_every_layer(name, merge, layer):
    """All five workloads, every layer, in lock-step with the oracle in the launch configuration the
    benchmark times (all layers in one cache, two scratch sets): attention outputs within 2e-2, the
    library's own scores within 1e-3 relative on every evicting block, and under the oracle's
    scores kept sets, merge plans, token indices and weights bit-exact, rows within one bf16 ulp."""
    wl = get_workload(name)
    cache = K.Cache(wl.n_layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk,
                    wl.segments, merge=merge, scratch_sets=min(2, wl.n_layers), device=DEV)
    qb, kb, vb = layer_inputs(wl, layer)
    stats = {}
    U.lockstep_layer(wl, layer, cache, qb, kb, vb, merge, stats=stats)
    print(name, "layer", layer, "merge", merge, stats, flush=True)
    assert stats["scored_blocks"] == sum(1 for t0, n in chunk_ranges(wl.n_tokens, wl.chunk) if t0 + n > wl.budget)
    assert stats["score_rel"] <= U.SCORE_RTOL
    if merge:
        assert stats["merged"] > 0
    cache.close()


@pytest.mark.parametrize("name,max_layers", [("tiny", 99), ("single_image", 99), ("tiled_image", 99),
                                             ("video", 2), ("long_video", 1)])   # the large ones: their first layers
def test_free_running_overlap_with_the_oracle(name, max_layers):
    """Free-running report: the library runs the whole prefill on its OWN scores, the oracle on its
    own; nothing is re-synchronised.  Scores agree to about 1e-5, so the two only part where two
    candidates are nearly tied, and a different choice then changes the cache both go on with.
    Reported per KV head: Jaccard overlap of the final kept token sets; and the error of the last
    block's attention output, which has seen every difference before it."""
    wl = get_workload(name)
    cache = K.Cache(wl.n_layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk,
                    wl.segments, merge=True, scratch_sets=min(2, wl.n_layers), device=DEV)
    ranges = chunk_ranges(wl.n_tokens, wl.chunk)
    overlaps, out_errs = [], []
    for layer in range(min(wl.n_layers, max_layers)):
        qb, kb, vb = layer_inputs(wl, layer)
        qt, kt, vt = (U.bits_to_torch(x) for x in (qb, kb, vb))
        q64, k64, v64 = (bf16_bits_to_f32(x).astype(np.float64) for x in (qb, kb, vb))
        out = None
        for t0, n in ranges:
            out = cache.prefill_chunk(layer, t0, qt[t0:t0 + n], kt[t0:t0 + n], vt[t0:t0 + n])
            cache.compact(layer)
        oc, recs = O.prefill_layer(q64, k64, v64, wl.chunk, wl.budget, wl.segments, True)
        k, v, idx, w, count, nxt = cache.decode_ready(layer)
        assert count == oc.count and nxt == wl.n_tokens
        idx = idx.cpu().numpy()
        overlaps += [U.jaccard(idx[hk, :count], oc.idx[hk]) for hk in range(wl.n_kv_heads)]
        out_errs.append(U.out_rel_err(U.torch_bf16_to_f64(out), recs[-1]["out"]))
    print("free-running %s: kept-set Jaccard per head min %.4f mean %.4f; last-block out rel err max %.4g"
          % (name, min(overlaps), float(np.mean(overlaps)), max(out_errs)), flush=True)
    assert min(overlaps) >= FREE_RUNNING_JACCARD_FLOOR
    assert max(out_errs) <= FREE_RUNNING_OUT_TOL
    cache.close()


def test_odd_sizes_lockstep():
    """Block and budget that are not multiples of any tile, three segments, two visual."""
    segs = (Segment(0, 7, 0), Segment(7, 3 * 5 * 9, 1, 5, 9, 3, 1), Segment(142, 11, 0),
            Segment(153, 2 * 6 * 6, 1, 6, 6, 2, 0), Segment(225, 20, 0))
    wl = Workload("odd", 1, 6, 2, 64, 37, 61, segs, "plane")
    qb, kb, vb = layer_inputs(wl, 0, seed0=3)
    for merge in (False, True):
        cache = K.Cache(1, 6, 2, 64, 61, 37, segs, merge=merge, device=DEV)
        U.lockstep_layer(wl, 0, cache, qb, kb, vb, merge)
        cache.close()


@pytest.mark.parametrize("shape", [-1, 2])
@pytest.mark.parametrize("hq,hkv,d,c,n", [(2, 2, 128, 200, 55), (2, 1, 128, 700, 324), (2, 1, 128, 700, 325), (4, 2, 64, 100, 413),
                                          (2, 1, 64, 1500, 548), (2, 1, 64, 1500, 549),
                                          # 8, 16 and 24 rows per thread, and one key more
                                          (2, 2, 128, 200, 56), (2, 2, 128, 200, 57), (2, 1, 128, 400, 112), (2, 1, 128, 400, 113),
                                          (2, 1, 128, 700, 68), (2, 1, 128, 700, 69), (4, 2, 64, 100, 412), (2, 1, 64, 700, 324),
                                          (2, 1, 64, 700, 325), (2, 1, 64, 1500, 36), (2, 1, 64, 1500, 37)])
def test_keydiff_scored_by_the_compaction_edges(hq, hkv, d, c, n, shape):
    """Scores by the keys alone beside the attention (shape -1: the split-key shapes) and inside the compaction launch (shape 2):
    each of the up to 32 rows per thread that this is built for, and the first heads that are too large for both."""
    assert _rows_of_a_workgroup(n, hq) == 32
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, c, 600, seed=c + n, keydiff=True, attention_shape=shape)
    assert err <= U.OUT_TOL, err
    scores_gpu, keep, _ = cache.debug_last(0)
    got = scores_gpu.cpu().numpy().astype(np.float64)
    assert np.abs(got - scores_ref).max() <= 2e-5
    tok = np.concatenate([oc.idx, np.broadcast_to(np.arange(c, c + n), (hkv, n))], axis=1)
    for hk in range(hkv):
        assert np.array_equal(keep.cpu().numpy()[hk].astype(bool), O.select_keep(scores_gpu.cpu().numpy()[hk], tok[hk], c))
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,c,n", [
    # nothing cached, one key of the block evicted; ten KV heads; the most candidates; two row tiles per workgroup; as many
    # 32-row workgroups as CUs with the scoring ones, and one more
    (4, 2, 128, 0, 2), (4, 2, 64, 1, 1), (20, 10, 64, 300, 33), (4, 2, 128, 900, 124), (4, 2, 64, 1900, 148), (28, 4, 128, 512, 512),
    (31, 1, 128, 512, 256), (32, 8, 128, 512, 256)])
def test_keys_scored_beside_the_attention(hq, hkv, d, c, n):
    """Scores by the keys alone from the attention launch of the split-key shapes, and from the compaction launch behind the
    128-row shape: the same bits."""
    scores = []
    for shape in (-1, 2):
        cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, c, n, max(c, n - 1, 1), 600, seed=c + 3 * n, keydiff=True,
                                                        attention_shape=shape)
        assert err <= U.OUT_TOL, err
        scores.append(cache.debug_last(0)[0].cpu().numpy().copy())
        assert np.abs(scores[-1].astype(np.float64) - scores_ref).max() <= 2e-5
        cache.close()
    assert np.array_equal(scores[0].view(np.uint32), scores[1].view(np.uint32))


def test_key_scores_of_grouped_and_single_launches():
    """Six layers of 184 workgroups at d 64: scored beside the attention one layer at a time, in the compaction together."""
    layers, hq, hkv, d, c, n = 6, 16, 4, 64, 1111, 333
    rng = np.random.default_rng(6)
    data = [tuple(U.bits_to_torch(_rand_bits(rng, (n, h, d))) for h in (hq, hkv, hkv)) for _ in range(layers)]
    rows = U.bits_to_torch(_rand_bits(rng, (2, hkv, c, d)))
    results = []
    for grouped in (False, True):
        cache = K.Cache(layers, hq, hkv, d, c, n, [Segment(0, 4000, 0)], merge=False, scratch_sets=layers, device=DEV)
        outs = [torch.empty_like(q) for q, _, _ in data]
        for l in range(layers):
            k, v, idx, w, _, _ = cache.decode_ready(l)
            k.copy_(rows[0]); v.copy_(rows[1]); w.fill_(1.0)
            idx.copy_(torch.arange(c, device=DEV, dtype=torch.int32).expand(hkv, c))
            cache.set_state(l, c, c)
        if grouped:
            K.Prefill(cache, layers).block(c, lambda l: data[l], lambda l: outs[l], None, True)
        else:
            for l in range(layers):
                cache.prefill_chunk_keydiff(l, c, *data[l], out=outs[l])
                cache.compact(l)
        scores = [cache.debug_last(l)[0] for l in range(layers)]
        results.append([x.clone() for l in range(layers) for x in cache.decode_ready(l)[:4]] + [x.clone() for x in scores] + outs)
        cache.close()
    for a, b in zip(*results):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("d,c,n,budget,t0,levels", [
    (64, 700, 324, 700, 700, 5),          # 1024 candidates, one per thread; hundreds of equal scores at the threshold
    (128, 700, 325, 650, 30000, 40),      # one more; a token table with an entry per token of a long prefix
    (64, 900, 1100, 1000, 60000, 9),      # a prefix too long for that: the hash table
    (128, 3000, 1096, 3000, 3000, 3),     # 4096 candidates, the most with source lists in LDS
    (64, 3000, 1097, 3100, 90000, 100000)])   # one more
def test_compaction_edges(d, c, n, budget, t0, levels):
    """Selection, merge plan and rows at the edges of the compaction kernel's ranges: candidates per thread,
    more equal scores than a wave can rank, the two kinds of token table."""
    hkv, gh, gw = 2, 16, 16
    rng = np.random.default_rng(c + n)
    planes = (t0 + n) // (gh * gw) + 1
    segs = (Segment(0, planes * gh * gw, 1, gh, gw, planes, 1),)
    cache = K.Cache(1, hkv, hkv, d, budget, max(n, c), segs, merge=True, device=DEV)
    oc = O.LayerCache(hkv, d, budget, segs, True)
    kb0, vb0 = _rand_bits(rng, (c, hkv, d)), _rand_bits(rng, (c, hkv, d))
    k0, v0 = O.bf16_bits_to_f64(kb0), O.bf16_bits_to_f64(vb0)
    keep = min(c, budget)
    # cached tokens from the last few thousand before the block, in any slot order
    oc.idx = np.stack([rng.choice(np.arange(max(0, t0 - 4 * c), t0), size=keep, replace=False) for _ in range(hkv)])
    oc.w = rng.integers(1, 4, size=(hkv, keep))
    oc.K, oc.V, oc.count = k0[:keep].transpose(1, 0, 2).copy(), v0[:keep].transpose(1, 0, 2).copy(), keep
    U.upload_state(cache, 0, oc)
    cache.set_state(0, keep, t0)
    qb, kb, vb = _rand_bits(rng, (n, hkv, d)), _rand_bits(rng, (n, hkv, d)), _rand_bits(rng, (n, hkv, d))
    scores = (rng.integers(0, levels, size=(hkv, keep + n)).astype(np.float32) + 1) / 7
    cache.prefill_chunk(0, t0, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
    cache.compact(0, torch.from_numpy(scores).to(DEV))
    rec = oc.compact(t0, O.bf16_bits_to_f64(kb), O.bf16_bits_to_f64(vb), scores)
    used, kept, dst = cache.debug_last(0)
    assert np.array_equal(used.cpu().numpy(), scores)
    assert np.array_equal(kept.cpu().numpy().astype(bool), rec["keep"])
    assert np.array_equal(dst.cpu().numpy().astype(np.int64), rec["dst"])
    assert U.compare_state(cache, 0, oc) > 0
    cache.close()


def _compact_on_given_scores(d, c, n, budget, t0, segs, tokens, scores):
    """A cache preloaded with `tokens` [2, c], one block of n tokens, a compaction on `scores`: the caches of the library
    and of the oracle, kept set, merge plan, token indices, weights and rows compared."""
    hkv = 2
    rng = np.random.default_rng(c + n)
    cache = K.Cache(1, hkv, hkv, d, budget, n, segs, merge=True, device=DEV)
    oc = O.LayerCache(hkv, d, budget, segs, True)
    oc.idx, oc.count = np.asarray(tokens, dtype=np.int64), c
    oc.w = rng.integers(1, 4, size=(hkv, c))
    oc.K, oc.V = (O.bf16_bits_to_f64(_rand_bits(rng, (hkv, c, d))) for _ in range(2))
    U.upload_state(cache, 0, oc)
    cache.set_state(0, c, t0)
    qb, kb, vb = (_rand_bits(rng, (n, hkv, d)) for _ in range(3))
    cache.prefill_chunk(0, t0, U.bits_to_torch(qb), U.bits_to_torch(kb), U.bits_to_torch(vb))
    cache.compact(0, torch.from_numpy(scores).to(DEV))
    rec = oc.compact(t0, O.bf16_bits_to_f64(kb), O.bf16_bits_to_f64(vb), scores)
    used, kept, dst = cache.debug_last(0)
    assert np.array_equal(used.cpu().numpy(), scores)
    assert np.array_equal(kept.cpu().numpy().astype(bool), rec["keep"])
    assert np.array_equal(dst.cpu().numpy().astype(np.int64), rec["dst"])
    merged = U.compare_state(cache, 0, oc)
    return cache, merged


@pytest.mark.parametrize("d,c,n", [(64, 3, 1), (128, 400, 112), (64, 400, 113), (128, 700, 324), (64, 700, 325), (128, 1500, 548),
                                   (64, 1500, 549), (128, 1900, 1172), (64, 1900, 1173)])
@pytest.mark.parametrize("t0", [2000, 70000])                 # the two kinds of token table
def test_compaction_workgroup_sizes(d, c, n, t0):
    """The smallest head, one candidate per thread of 512 and one more, the most candidates that 512 threads take and one
    more, two per thread of 1024 and one more, three and one more."""
    planes = (t0 + n) // 256 + 1
    rng = np.random.default_rng(t0 + c + n)
    tokens = np.stack([rng.choice(np.arange(t0 - min(t0, 2 * c), t0), size=c, replace=False) for _ in range(2)])
    scores = (rng.integers(0, 50, size=(2, c + n)).astype(np.float32) + 1) / 7
    cache, merged = _compact_on_given_scores(d, c, n, c, t0, (Segment(0, planes * 256, 1, 16, 16, planes, 1),), tokens, scores)
    assert merged > 0 or c < 100
    cache.close()


@pytest.mark.parametrize("d,c,n", [(64, 60, 4), (128, 400, 112), (64, 400, 113), (128, 1500, 549)])   # owners plan up to 512, any thread beyond
@pytest.mark.parametrize("t0", [2000, 70000])                 # the two kinds of token table
@pytest.mark.parametrize("first", ["text", "visual"])
def test_merge_plan_of_several_segments(d, c, n, t0, first):
    """Evicted tokens in the first segment, in later ones and in text; neighbours cached and in the block, in still and moving
    pictures, up to the segment's edges."""
    head = (Segment(0, 24, 0),) if first == "text" else (Segment(0, 24, 1, 4, 6, 1, 0),)
    still = Segment(24, (t0 - c // 2) // 64 * 64, 1, 8, 8, (t0 - c // 2) // 64, 0)
    at = 24 + still.n_tokens + 9
    planes = (t0 + n - at) // 30 + 1
    segs = head + (still, Segment(at - 9, 9, 0), Segment(at, planes * 30, 1, 5, 6, planes, 1), Segment(at + planes * 30, 1000, 0))
    rng = np.random.default_rng(t0 + c + n)
    tokens = np.stack([np.r_[np.arange(12), rng.choice(np.arange(max(12, t0 - 2 * c), t0), size=c - 12, replace=False)] for _ in range(2)])
    scores = (rng.integers(0, 50, size=(2, c + n)).astype(np.float32) + 1) / 7
    cache, merged = _compact_on_given_scores(d, c, n, c, t0, segs, tokens, scores)
    assert merged > 0 or c < 100
    cache.close()


@pytest.mark.parametrize("total", [512, 1024, 1025, 2048, 2049, 3072, 3073, 4096, 4097])
def test_sums_of_many_partial_arrays(total):
    """Own scores summed by the compaction from more partial arrays than its loads in flight, at the edges of its passes."""
    n, hq, hkv, d = 330, 8, 1, 64
    cache, oc, err, scores_ref, _ = _attention_case(hq, hkv, d, total - n, n, total - 1, 512, seed=total)
    assert err <= U.OUT_TOL, err
    U.check_scores(cache.debug_last(0)[0].cpu().numpy(), scores_ref, n * hq)
    cache.close()


@pytest.mark.parametrize("d,c,n,budget,t0", [(128, 2048, 1024, 2048, 2048),     # the bench shape
                                             (64, 1536, 512, 1536, 1536), (64, 512, 256, 512, 700), (64, 4100, 200, 4100, 5000)])
@pytest.mark.parametrize("kind", ["equal", "half_zero", "zeros"])
def test_selection_among_equal_scores(kind, d, c, n, budget, t0):
    """Hundreds of equal scores around the threshold, all of them or beside ordinary ones: as many are kept as the budget
    says, the lower token indices."""
    rng = np.random.default_rng(c)
    gh, gw = 16, 16
    planes = (t0 + n) // (gh * gw) + 1
    tokens = np.stack([rng.permutation(t0)[:c] for _ in range(2)])
    scores = np.full((2, c + n), 0.75 if kind == "equal" else 0.0, dtype=np.float32)
    if kind == "half_zero":
        some = rng.permutation(c + n)[:(c + n) // 2]
        scores[:, some] = 4 * rng.random((2, len(some)), dtype=np.float32)
    cache, merged = _compact_on_given_scores(d, c, n, budget, t0, (Segment(0, planes * gh * gw, 1, gh, gw, planes, 1),), tokens, scores)
    assert merged > 0
    cache.close()


@pytest.mark.parametrize("d,c,n,t0", [(64, 700, 324, 700),         # the table has an entry per token before the block
                                      (128, 900, 1100, 60000)])     # a hash table
def test_cached_tokens_that_the_block_does_not_follow(d, c, n, t0):
    """A cache written from outside (kvp_set_state) whose token indices are not all below the block: they compete like
    any other, and the compaction stays inside its memory."""
    rng = np.random.default_rng(t0)
    gh, gw = 16, 16
    planes = (t0 + n) // (gh * gw) + 1
    n_vis = planes * gh * gw
    segs = (Segment(0, n_vis, 1, gh, gw, planes, 1), Segment(n_vis, 100000, 0))
    tokens = np.stack([rng.permutation(t0)[:c] for _ in range(2)])
    late = rng.permutation(c)[:c // 3]
    tokens[:, late] = n_vis + rng.permutation(100000)[:len(late)]          # text: nothing to merge, on either side
    scores = rng.random((2, c + n), dtype=np.float32)
    tokens[:, late[0]], scores[:, late[0]] = -1, 2.0                       # (kept: the oracle has no place for an evicted one)
    cache, merged = _compact_on_given_scores(d, c, n, c, t0, segs, tokens, scores)
    assert merged > 0
    cache.close()


@pytest.mark.parametrize("t0", [1000, 60000])                 # the two kinds of token table
@pytest.mark.parametrize("copies", [2, 40, 300])
def test_cached_tokens_that_repeat(copies, t0):
    """A cache written from outside whose token indices repeat is no valid state: the compaction still ends, stays inside
    its memory, keeps what is ordinary about the case, and merges one of the slots that share a token."""
    hkv, d, c, n = 2, 64, 1000, 300
    rng = np.random.default_rng(copies)
    gh, gw = 16, 16
    planes = (t0 + n) // (gh * gw) + 1
    segs = (Segment(0, planes * gh * gw, 1, gh, gw, planes, 1),)
    bits = [_rand_bits(rng, shape) for shape in [(hkv, c, d)] * 2 + [(n, hkv, d)] * 3]
    at = 8 * gw + 8                                           # a token with five neighbours before the block
    first = [at - 1, at + 1, at - gw, at + gw, at + gh * gw]
    others = np.setdiff1d(np.arange(t0), first + [at])
    tok = np.concatenate([first, np.full(copies, at), rng.permutation(others)[:c]])[:c]
    assert len(tok) == c
    for kind in ("evicted", "threshold"):
        scores = 0.5 + rng.random((hkv, c + n), dtype=np.float32) / 4
        scores[:, :5] = 1.0
        if kind == "evicted":
            scores[:, 5:5 + copies] = 0.25
        else:                     # room for half of the copies, ten free slots for copies / 2 + 10 rows of the block
            scores[:, 5:5 + copies] = 0.5
            scores[:, c - 10:] = 0.25
            scores[:, c:c + copies // 2 + 10] = 0.9
        cache = K.Cache(1, hkv, hkv, d, c, n, segs, merge=True, device=DEV)
        k, v, idx, w, _, _ = cache.decode_ready(0)
        k.copy_(U.bits_to_torch(bits[0]))
        v.copy_(U.bits_to_torch(bits[1]))
        idx.copy_(torch.from_numpy(np.stack([tok] * hkv).astype(np.int32)))
        w.fill_(1.0)
        cache.set_state(0, c, t0)
        cache.prefill_chunk(0, t0, *(U.bits_to_torch(x) for x in bits[2:]))
        cache.compact(0, torch.from_numpy(scores).to(DEV))
        torch.cuda.synchronize()
        assert cache.guards_intact()
        _, kept, dst = (x.cpu().numpy() for x in cache.debug_last(0))
        idx, w = idx.cpu().numpy(), w.cpu().numpy()
        order = ~np.concatenate([tok, np.arange(t0, t0 + n)]).astype(np.uint32)
        for hk in range(hkv):
            keys = (scores[hk].view(np.uint32).astype(np.uint64) << np.uint64(32)) | order.astype(np.uint64)
            want = keys >= np.sort(keys)[n]                   # the c largest of c + n, and what equals the smallest of them
            assert np.array_equal(kept[hk].astype(bool), want)
            assert np.array_equal(idx[hk][want[:c]], tok[want[:c]])                    # kept slots keep their tokens
            assert sorted(idx[hk][~want[:c]]) == (t0 + np.flatnonzero(want[c:]))[:(~want[:c]).sum()].tolist()
            assert (w[hk] >= 1).all() and w[hk].max() <= 7
            if kind == "evicted":
                copies_of = np.flatnonzero(tok == at)
                evicted = copies_of[~want[copies_of]]
                assert (dst[hk][evicted] >= 0).sum() == 1 and set(dst[hk][evicted]) <= {-1, 0, 1, 2, 3, 4}
        cache.close()


@pytest.mark.parametrize("merge", [False, True])
@pytest.mark.parametrize("hkv,layers", [(2, 1), (8, 6)])
def test_running_totals(merge, hkv, layers):
    """Every compaction adds what its plan says to the counters."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(hkv)
    cache = K.Cache(layers, hkv, hkv, 64, 96, 64, [K.KvpSegment(0, 800, K.KVP_VISUAL, 10, 10, 8, 1)], merge=merge, scratch_sets=layers,
                    device=DEV)
    want = [0, 0, 0, 0]
    for t0 in range(0, 448, 64):
        for layer in range(layers):
            draw = lambda: torch.randn((64, hkv, 64), generator=gen, device="cuda", dtype=torch.bfloat16)
            cache.prefill_chunk(layer, t0, draw(), draw(), draw())
        count = min(t0, 96)
        cache.compact_layers(0, layers)
        if count + 64 <= 96:
            continue
        for layer in range(layers):
            _, keep, dst = cache.debug_last(layer)
            merged = (dst >= 0) & (keep == 0)
            want[0] += hkv
            want[1] += int(keep[:, count:].sum())
            want[2] += sum(len(torch.unique(dst[h][merged[h]])) for h in range(hkv))
            want[3] += int(merged.sum())
    totals = cache.totals()
    assert [totals[name] for name in K.binding.TOTALS] == want
    assert want[1] > 0 and (want[3] > 0) == merge
    cache.close()


def test_maximum_candidates_lockstep():
    """budget + block at the library's limit (8192 candidates per head): the select kernel's
    eight-candidates-per-thread shape, its largest LDS layout, 2048-row blocks."""
    segs = (Segment(0, 16 * 16 * 47, 1, 16, 16, 47, 1), Segment(16 * 16 * 47, 256, 0))
    wl = Workload("max", 1, 2, 2, 64, 2048, 6144, segs, "shared")
    assert wl.n_tokens == 6 * 2048 and wl.budget + wl.chunk == 8192
    qb, kb, vb = layer_inputs(wl, 0, seed0=11)
    cache = K.Cache(1, 2, 2, 64, wl.budget, wl.chunk, segs, merge=True, device=DEV)
    stats = {}
    U.lockstep_layer(wl, 0, cache, qb, kb, vb, True, stats=stats)
    assert stats["merged"] > 0
    cache.close()


@pytest.mark.parametrize("hq,hkv,d,chunk,budget,segs", [
    # one slot per head, one token per block: every block evicts exactly one candidate of two
    (2, 2, 64, 1, 1, (Segment(0, 3 * 3, 1, 3, 3, 1, 0), Segment(9, 4, 0))),
    # block larger than the budget: the very first block already evicts, with an empty cache
    (4, 2, 64, 48, 16, (Segment(0, 6 * 8 * 2, 1, 6, 8, 2, 1), Segment(96, 10, 0))),
    # text only: nothing can merge, merge on must equal merge off
    (4, 1, 128, 24, 40, (Segment(0, 100, 0),)),
    # a single-row, single-column grid per plane: only temporal neighbours exist
    (2, 1, 64, 5, 7, (Segment(0, 23, 1, 1, 1, 23, 1),)),
])
def test_degenerate_shapes_lockstep(hq, hkv, d, chunk, budget, segs):
    wl = Workload("degenerate", 1, hq, hkv, d, chunk, budget, segs, "plane")
    qb, kb, vb = layer_inputs(wl, 0, seed0=5)
    for merge in (False, True):
        cache = K.Cache(1, hq, hkv, d, budget, chunk, segs, merge=merge, device=DEV)
        U.lockstep_layer(wl, 0, cache, qb, kb, vb, merge)
        cache.close()


def test_structure_aligned_blocks_and_bulk_first_pass_lockstep():
    """Blocks cut at frame boundaries, of different lengths, after a first block that fills the
    whole budget in one causal pass (Sec. 3.1 and the hybrid execution of Sec. 4.3): any block
    length up to chunk_max goes through the same kernels."""
    gh, gw, frames, n_text = 14, 14, 24, 40                     # 196-token frames
    per = gh * gw
    segs = (Segment(0, per * frames, 1, gh, gw, frames, 1), Segment(per * frames, n_text, 0))
    budget = 4 * per                                            # 784 = four frames
    wl = Workload("aligned", 1, 8, 2, 128, budget, budget, segs, "shared")
    # bulk first pass of `budget` tokens, then blocks of one, three, two ... frames, then the text
    lengths = [4 * per, per, 3 * per, 2 * per, 4 * per, per, 2 * per, 3 * per, 4 * per, n_text]
    assert sum(lengths) == wl.n_tokens
    blocks, t0 = [], 0
    for n in lengths:
        blocks.append((t0, n))
        t0 += n
    qb, kb, vb = layer_inputs(wl, 0, seed0=17)
    for merge in (False, True):
        cache = K.Cache(1, 8, 2, 128, budget, budget, segs, merge=merge, device=DEV)
        stats = {}
        U.lockstep_layer(wl, 0, cache, qb, kb, vb, merge, stats=stats, blocks=blocks)
        assert merge == (stats["merged"] > 0)
        cache.close()


def test_budget_at_least_prefix_is_full_attention():
    """Alg. 1 line 8 never fires: the GPU path must equal plain causal attention."""
    wl = get_workload("tiny")
    qb, kb, vb = layer_inputs(wl, 0)
    q64, k64, v64 = (bf16_bits_to_f32(x).astype(np.float64) for x in (qb, kb, vb))
    n_tok = wl.n_tokens
    cache = K.Cache(1, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, 1024, 96, wl.segments, merge=True, device=DEV)
    qt, kt, vt = (U.bits_to_torch(x) for x in (qb, kb, vb))
    outs = []
    for t0, n in chunk_ranges(n_tok, 96):
        outs.append(cache.prefill_chunk(0, t0, qt[t0:t0 + n], kt[t0:t0 + n], vt[t0:t0 + n]))
        cache.compact(0)
    out = U.torch_bf16_to_f64(torch.cat(outs))
    ref, _ = O.attend_chunk(q64, k64.transpose(1, 0, 2), v64.transpose(1, 0, 2), 0)
    assert U.out_rel_err(out, ref) <= U.OUT_TOL
    k, v, idx, w, count, _ = cache.decode_ready(0)
    assert count == n_tok
    assert np.array_equal(idx[:, :n_tok].cpu().numpy(), np.broadcast_to(np.arange(n_tok), (wl.n_kv_heads, n_tok)))
    assert np.array_equal(U.torch_to_bits(k[:, :n_tok]), kb.transpose(1, 0, 2))
    assert np.array_equal(U.torch_to_bits(v[:, :n_tok]), vb.transpose(1, 0, 2))
    assert bool((w[:, :n_tok] == 1).all())
    cache.close()


@pytest.mark.parametrize("name", ["tiled_image", "long_video"])
def test_free_running_invariants(name):
    """The whole prefill on the GPU's own scores, all layers: properties that hold at
    any size (Alg. 1 invariants, softmax rows summing to one, determinism)."""
    wl = get_workload(name)
    layers = list(range(wl.n_layers)) if name != "long_video" else [0, 1]
    results = []
    for rep in range(2):
        cache = K.Cache(wl.n_layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk,
                        wl.segments, merge=True, scratch_sets=2, device=DEV)
        final = {}
        for layer in layers:
            qb, kb, vb = layer_inputs(wl, layer)
            qt, kt, vt = (U.bits_to_torch(x) for x in (qb, kb, vb))
            seen = 0
            for t0, n in chunk_ranges(wl.n_tokens, wl.chunk):
                cache.prefill_chunk(layer, t0, qt[t0:t0 + n], kt[t0:t0 + n], vt[t0:t0 + n])
                c_before = min(wl.budget, seen)
                cache.compact(layer)
                seen += n
                if c_before + n > wl.budget:
                    sc, keep, dst = cache.debug_last(layer)
                    s = sc.sum(dim=1).cpu().numpy()
                    np.testing.assert_allclose(s, n * wl.group, rtol=1e-4)
                    assert int(keep.sum(dim=1).min()) == int(keep.sum(dim=1).max()) == wl.budget
                k, v, idx, w, count, nxt = cache.decode_ready(layer)
                assert count == min(wl.budget, seen) and nxt == seen
            idx = idx.cpu().numpy()
            w = w.cpu().numpy()
            for hk in range(wl.n_kv_heads):
                assert len(set(idx[hk].tolist())) == wl.budget and idx[hk].max() < wl.n_tokens and idx[hk].min() >= 0
                assert (w[hk] >= 1).all() and (w[hk] == np.round(w[hk])).all() and w[hk].sum() <= wl.n_tokens
            final[layer] = (idx.copy(), U.torch_to_bits(k).copy())
        results.append(final)
        cache.close()
    for layer in layers:      # two runs agree bit for bit: no atomics on floats anywhere
        assert np.array_equal(results[0][layer][0], results[1][layer][0])
        assert np.array_equal(results[0][layer][1], results[1][layer][1])


@pytest.mark.parametrize("name,sets,scoring", [
    ("tiled_image", 2, "own"), ("video", 2, "own"), ("tiled_image", 3, "own"), ("video", 4, "own"), ("tiled_image", 6, "own"),
    ("video", 5, "own"), ("video", 8, "own"), ("tiled_image", 7, "own"),
    ("tiled_image", 4, "proxy"), ("video", 8, "proxy"), ("tiled_image", 4, "keydiff"), ("video", 6, "keydiff"),
    ("long_video", 8, "own")])                      # the benchmark's shape and scratch sets, eight of its layers
def test_compaction_on_a_second_stream_changes_nothing(name, sets, scoring):
    """The whole prefill with every kvp_compact on a second stream (events between the streams, one
    pair per group of layers) must leave bit for bit the caches and outputs of the in-order run,
    whichever way the candidates are scored."""
    wl = get_workload(name)
    layers = min(wl.n_layers, max(6, sets))      # groups of sets / 2 layers; 5 and 7 make the set use irregular
    data = [tuple(U.bits_to_torch(x) for x in layer_inputs(wl, l)) for l in range(layers)]
    ranges = chunk_ranges(wl.n_tokens, wl.chunk)
    results = []
    for overlap in (False, True):
        cache = K.Cache(layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk, wl.segments,
                        merge=True, scratch_sets=sets if overlap else 1, device=DEV)
        driver = K.Prefill(cache, layers, overlap=overlap)
        outs = [torch.zeros((wl.chunk, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device=DEV)
                for _ in range(layers)]
        obs = None
        if scoring == "proxy":
            gen = torch.Generator(device=DEV).manual_seed(99)
            obs = [torch.randn((24, wl.n_q_heads, wl.head_dim), generator=gen, device=DEV).to(torch.bfloat16)
                   for _ in range(layers)]
        for t0, n in ranges:
            driver.block(t0, lambda l: tuple(x[t0:t0 + n] for x in data[l]), lambda l: outs[l][:n],
                         (lambda l: obs[l]) if obs is not None else None, scoring == "keydiff")
        driver.finish()
        torch.cuda.synchronize()
        state = []
        for l in range(layers):
            k, v, idx, w, count, nxt = cache.decode_ready(l)
            state.append((k[:, :count].clone(), v[:, :count].clone(), idx[:, :count].clone(), w[:, :count].clone(),
                          count, nxt, outs[l].clone()))
        results.append(state)
        cache.close()
    for a, b in zip(*results):
        assert a[4] == b[4] and a[5] == b[5]
        for x, y in zip(a[:4] + (a[6],), b[:4] + (b[6],)):
            assert torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x,
                               y.view(torch.int16) if y.dtype == torch.bfloat16 else y)


@pytest.mark.parametrize("name,layers,scoring", [("tiled_image", 8, "own"), ("video", 5, "own"), ("video", 16, "keydiff"),
                                                 ("video", 19, "own"), ("tiled_image", 8, "proxy"), ("video", 9, "proxy")])
def test_compact_layers_is_the_per_layer_compaction(name, layers, scoring):
    """A model runs its layers one after the other: kvp_prefill_chunk per layer while the block
    moves up the stack, then ONE kvp_compact_layers for all of them (grouped launches, 16 layers at
    a time; 19 layers make it a group of 16 and one of 3; in the five-layer case one layer is held a
    block behind, which makes the range inhomogeneous).  Scored by proxy queries or by the keys, the
    grouped run also puts the scoring passes off until that call (kvp_set_deferred_scoring), so they
    too go out for the whole range at once.  Caches and outputs must be those of the call-by-call
    order, bit for bit."""
    wl = get_workload(name)
    data = [tuple(U.bits_to_torch(x) for x in layer_inputs(wl, l)) for l in range(layers)]
    ranges = chunk_ranges(wl.n_tokens, wl.chunk)
    results = []
    for grouped in (False, True):
        cache = K.Cache(layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk, wl.segments,
                        merge=True, scratch_sets=layers if grouped else 1, device=DEV)
        outs = [torch.zeros((wl.chunk, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device=DEV)
                for _ in range(layers)]
        obs = None
        if scoring == "proxy":
            gen = torch.Generator(device=DEV).manual_seed(7)
            obs = [torch.randn((40, wl.n_q_heads, wl.head_dim), generator=gen, device=DEV).to(torch.bfloat16)
                   for _ in range(layers)]
        if grouped and scoring != "own":
            cache.set_deferred_scoring(1)
        lag = layers - 2 if name == "video" and layers == 5 else -1      # this layer gets its blocks one call late
        pending_lag = None
        for t0, n in ranges:
            for l in range(layers):
                if l == lag:
                    continue
                q, k, v = (x[t0:t0 + n] for x in data[l])
                if scoring == "keydiff":
                    cache.prefill_chunk_keydiff(l, t0, q, k, v, out=outs[l][:n])
                elif scoring == "proxy":
                    cache.prefill_chunk_proxy(l, t0, q, k, v, obs[l], out=outs[l][:n])
                else:
                    cache.prefill_chunk(l, t0, q, k, v, out=outs[l][:n])
                if not grouped:
                    cache.compact(l)
            if lag >= 0:
                if pending_lag is not None:
                    pt0, pn = pending_lag
                    q, k, v = (x[pt0:pt0 + pn] for x in data[lag])
                    cache.prefill_chunk(lag, pt0, q, k, v, out=outs[lag][:pn])
                    if not grouped:
                        cache.compact(lag)
                pending_lag = (t0, n)
            if grouped:
                if lag >= 0 and pending_lag == ranges[0]:        # the lagging layer has nothing pending yet
                    cache.compact_layers(0, lag)
                    cache.compact_layers(lag + 1, layers - lag - 1)
                else:
                    cache.compact_layers(0, layers)
        torch.cuda.synchronize()
        state = []
        for l in range(layers):
            k, v, idx, w, count, nxt = cache.decode_ready(l)
            state.append((k[:, :count].clone(), v[:, :count].clone(), idx[:, :count].clone(), w[:, :count].clone(),
                          count, nxt, outs[l].clone()))
        results.append(state)
        cache.close()
    for a, b in zip(*results):
        assert a[4] == b[4] and a[5] == b[5]
        for x, y in zip(a[:4] + (a[6],), b[:4] + (b[6],)):
            assert torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x,
                               y.view(torch.int16) if y.dtype == torch.bfloat16 else y)


@pytest.mark.parametrize("layers,hq,hkv,d,c,n,n_obs", [
    # three row splits of a key block per workgroup; two and then one; a last split of a single row tile more
    (16, 8, 8, 64, 700, 300, 75), (12, 8, 8, 64, 700, 300, 75), (16, 6, 2, 128, 1793, 256, 193)])
def test_grouped_proxy_scores_edges(layers, hq, hkv, d, c, n, n_obs):
    """Workgroups of a grouped scoring launch take several row splits in turn: the scores are those
    of the launches for one layer, bit for bit (and those are checked against the oracle)."""
    gen = torch.Generator(device=DEV).manual_seed(c + n_obs)
    draw = lambda *shape: torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16)
    data = [(draw(c + n, hq, d), draw(c + n, hkv, d), draw(c + n, hkv, d), draw(n_obs, hq, d)) for _ in range(layers)]
    scores = []
    for grouped in (False, True):
        cache = K.Cache(layers, hq, hkv, d, c, max(c, n), [Segment(0, c + n, 0)], scratch_sets=layers, device=DEV)
        cache.set_deferred_scoring(int(grouped))
        for t0, m in ((0, c), (c, n)):
            for l, (q, k, v, o) in enumerate(data):
                cache.prefill_chunk_proxy(l, t0, q[t0:t0 + m], k[t0:t0 + m], v[t0:t0 + m], o)
            cache.compact_layers(0, layers)
        scores.append([cache.debug_last(l)[0].clone() for l in range(layers)])
        cache.close()
    assert all(torch.equal(x, y) for x, y in zip(*scores))


def test_bench_launch_configuration_changes_nothing():
    """bench.py's default order at its own shape: everything in line on one stream, sixteen scratch
    sets, so that attention and compaction go out once per sixteen layers of long_video.  The first
    five blocks (two that only append, three that evict) of sixteen layers must leave the caches
    and outputs of the layer-by-layer order with one scratch set, bit for bit."""
    wl = get_workload("long_video")
    layers = 16
    data = [tuple(U.bits_to_torch(x) for x in layer_inputs(wl, l)) for l in range(layers)]
    ranges = chunk_ranges(wl.n_tokens, wl.chunk)[:5]
    results = []
    for sets in (1, 16):
        cache = K.Cache(layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk, wl.segments,
                        merge=True, scratch_sets=sets, device=DEV)
        driver = K.Prefill(cache, layers, overlap=False)
        outs = [torch.zeros((wl.chunk, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device=DEV)
                for _ in range(layers)]
        for t0, n in ranges:
            driver.block(t0, lambda l: tuple(x[t0:t0 + n] for x in data[l]), lambda l: outs[l][:n])
        driver.finish()
        torch.cuda.synchronize()
        state = []
        for l in range(layers):
            k, v, idx, w, count, nxt = cache.decode_ready(l)
            state.append((k[:, :count].clone(), v[:, :count].clone(), idx[:, :count].clone(), w[:, :count].clone(),
                          count, nxt, outs[l].clone()))
        results.append(state)
        cache.close()
    for a, b in zip(*results):
        assert a[4] == b[4] and a[5] == b[5]
        for x, y in zip(a[:4] + (a[6],), b[:4] + (b[6],)):
            assert torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x,
                               y.view(torch.int16) if y.dtype == torch.bfloat16 else y)


@pytest.mark.parametrize("scoring", ["own", "proxy", "keydiff"])
def test_layerwise_driver_matches_the_block_driver(scoring):
    """The two orders of calls of runtime.py, a whole block at once (Prefill) and layer by layer with
    one kvp_compact_layers per block (LayerwisePrefill, freshly allocated K and V per layer as a
    model would have them), leave the same caches and outputs bit for bit."""
    wl = get_workload("tiled_image")
    layers = wl.n_layers
    data = [tuple(U.bits_to_torch(x) for x in layer_inputs(wl, l)) for l in range(layers)]
    gen = torch.Generator(device=DEV).manual_seed(5)
    obs = [torch.randn((24, wl.n_q_heads, wl.head_dim), generator=gen, device=DEV).to(torch.bfloat16)
           for _ in range(layers)]
    ranges = chunk_ranges(wl.n_tokens, wl.chunk)
    results = []
    for layerwise in (False, True):
        cache = K.Cache(layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk, wl.segments,
                        merge=True, scratch_sets=layers, device=DEV)
        outs = [torch.zeros((wl.chunk, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device=DEV)
                for _ in range(layers)]
        if layerwise:
            driver = K.LayerwisePrefill(cache, layers)
            for t0, n in ranges:
                for l in range(layers):
                    q, k, v = (x[t0:t0 + n].clone() for x in data[l])
                    driver.layer(l, t0, q, k, v, out=outs[l][:n], q_obs=obs[l] if scoring == "proxy" else None,
                                 keydiff=scoring == "keydiff")
                    del q, k, v
                driver.end_block()
        else:
            driver = K.Prefill(cache, layers)
            for t0, n in ranges:
                driver.block(t0, lambda l: tuple(x[t0:t0 + n] for x in data[l]), lambda l: outs[l][:n],
                             (lambda l: obs[l]) if scoring == "proxy" else None, scoring == "keydiff")
            driver.finish()
        torch.cuda.synchronize()
        state = []
        for l in range(layers):
            k, v, idx, w, count, nxt = cache.decode_ready(l)
            state.append((k[:, :count].clone(), v[:, :count].clone(), idx[:, :count].clone(), w[:, :count].clone(),
                          count, nxt, outs[l].clone()))
        results.append(state)
        cache.close()
    for a, b in zip(*results):
        assert a[4] == b[4] and a[5] == b[5]
        for x, y in zip(a[:4] + (a[6],), b[:4] + (b[6],)):
            assert torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x,
                               y.view(torch.int16) if y.dtype == torch.bfloat16 else y)


@pytest.mark.parametrize("streams", [1, 2])
@pytest.mark.parametrize("kind", ["one_out", "chain"])
def test_block_driver_with_layers_that_depend_on_each_other(kind, streams):
    """kvp_prefill_block over layers that share one output buffer, or whose queries are the output of the layer before:
    caches and outputs are those of the calls one by one."""
    wl = get_workload("tiled_image")
    layers, hq, hkv, d = 6, wl.n_q_heads, wl.n_kv_heads, wl.head_dim
    data = [tuple(U.bits_to_torch(x) for x in layer_inputs(wl, l)) for l in range(layers)]
    ranges = chunk_ranges(wl.n_tokens, wl.chunk)[:6]                  # two that append, four that evict
    results = []
    for grouped in (False, True):
        cache = K.Cache(layers, hq, hkv, d, wl.budget, wl.chunk, wl.segments, merge=True, scratch_sets=4, device=DEV)
        outs = [torch.zeros((wl.chunk, hq, d), dtype=torch.bfloat16, device=DEV) for _ in range(layers)]
        if kind == "one_out":
            outs = [outs[0]] * layers
        driver = K.Prefill(cache, layers, overlap=streams == 2)
        seen = []
        for t0, n in ranges:
            def qkv(l):
                q, k, v = (x[t0:t0 + n] for x in data[l])
                return (outs[l - 1][:n] if kind == "chain" and l else q), k, v
            if grouped:
                driver.block(t0, qkv, lambda l: outs[l][:n])
            else:
                for l in range(layers):
                    cache.prefill_chunk(l, t0, *qkv(l), out=outs[l][:n])
                    cache.compact(l)
            seen.append(outs[-1].clone())
        driver.finish()
        for l in range(layers):
            k, v, idx, w, count, _ = cache.decode_ready(l)
            seen += [k[:, :count].clone(), v[:, :count].clone(), idx[:, :count].clone(), w[:, :count].clone()]
        torch.cuda.synchronize()
        results.append(seen)
        cache.close()
    bits = lambda t: t.view(torch.int16) if t.dtype == torch.bfloat16 else t
    assert all(torch.equal(bits(x), bits(y)) for x, y in zip(*results))


def test_real_cache_refuses_null_tensors():
    """A cache on a live allocation (not a dry run) returns KVP_EINVAL for a null tensor before it
    enqueues anything, and stays usable."""
    wl = get_workload("tiny")
    cache = K.Cache(1, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk, wl.segments, device=DEV)
    qb, kb, vb = layer_inputs(wl, 0)
    qt, kt, vt = (U.bits_to_torch(x)[:8].contiguous() for x in (qb, kb, vb))
    out = torch.empty_like(qt)
    ptrs = [qt.data_ptr(), kt.data_ptr(), vt.data_ptr(), out.data_ptr()]
    for hole in range(4):
        args = list(ptrs)
        args[hole] = 0
        assert K.kvp_prefill_chunk(cache.handle, 0, 0, 8, *args) == K.KVP_EINVAL
    assert K.kvp_decode_step(cache.handle, 0, 0, kt.data_ptr(), vt.data_ptr(), 1, out.data_ptr()) == K.KVP_EINVAL
    rc, vw = K.kvp_decode_ready(cache.handle, 0)
    assert rc == K.KVP_OK and (vw.count, vw.next_token) == (0, 0)          # nothing moved
    assert K.kvp_prefill_chunk(cache.handle, 0, 0, 8, *ptrs) == K.KVP_OK
    assert K.kvp_compact(cache.handle, 0) == K.KVP_OK
    torch.cuda.synchronize()
    cache.close()


@pytest.mark.parametrize("name,stop_after", [("tiny", 4), ("tiled_image", 5)])
def test_snapshot_restore_continue_is_bit_identical(name, stop_after):
    """Checkpoint and resume: the cache is the resumable state.  Run some blocks, copy out
    (K, V, token index, weight, count, next token) of every layer, free the cache, create a new one
    on a new buffer, write the copies back through the kvp_decode_ready pointers, declare them with
    kvp_set_state and go on: every later output and the final caches must equal, bit for bit,
    those of the run that was never interrupted."""
    wl = get_workload(name)
    layers = min(wl.n_layers, 3)
    data = [tuple(U.bits_to_torch(x) for x in layer_inputs(wl, l)) for l in range(layers)]
    ranges = chunk_ranges(wl.n_tokens, wl.chunk)

    def make():
        return K.Cache(layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk, wl.segments,
                       merge=True, device=DEV)

    def run(cache, blocks):
        outs = []
        for t0, n in blocks:
            for l in range(layers):
                q, k, v = (x[t0:t0 + n] for x in data[l])
                outs.append(cache.prefill_chunk(l, t0, q, k, v).clone())
                cache.compact(l)
        return outs

    def state(cache):
        st = []
        for l in range(layers):
            k, v, idx, w, count, nxt = cache.decode_ready(l)
            st.append((k[:, :count].clone(), v[:, :count].clone(), idx[:, :count].clone(), w[:, :count].clone(), count, nxt))
        return st

    straight = make()
    outs_a = run(straight, ranges)
    final_a = state(straight)
    straight.close()

    first = make()
    run(first, ranges[:stop_after])
    snap = state(first)
    torch.cuda.synchronize()
    first.close()
    del first
    second = make()
    for l, (k, v, idx, w, count, nxt) in enumerate(snap):
        k2, v2, idx2, w2, _, _ = second.decode_ready(l)
        k2[:, :count] = k
        v2[:, :count] = v
        idx2[:, :count] = idx
        w2[:, :count] = w
        second.set_state(l, count, nxt)
    outs_b = run(second, ranges[stop_after:])
    final_b = state(second)
    second.close()

    bits = lambda t: t.view(torch.int16) if t.dtype == torch.bfloat16 else t
    tail = outs_a[stop_after * layers:]
    assert len(tail) == len(outs_b)
    for a, b in zip(tail, outs_b):
        assert torch.equal(bits(a), bits(b))
    for a, b in zip(final_a, final_b):
        assert a[4] == b[4] and a[5] == b[5]
        for x, y in zip(a[:4], b[:4]):
            assert torch.equal(bits(x), bits(y))


def test_second_stream_with_freshly_allocated_blocks():
    """With compactions on the side stream a block's K and V are read after Prefill.block has
    returned.  A caller that allocates them per block and drops them at once must still get the
    in-order result: the driver keeps them alive (and out of the allocator's hands) until the
    side stream is done with them."""
    wl = get_workload("tiled_image")
    layers = 4
    host = [layer_inputs(wl, l) for l in range(layers)]
    ranges = chunk_ranges(wl.n_tokens, wl.chunk)
    results = []
    for overlap in (False, True):
        cache = K.Cache(layers, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.budget, wl.chunk, wl.segments,
                        merge=True, scratch_sets=4 if overlap else 1, device=DEV)
        driver = K.Prefill(cache, layers, overlap=overlap)
        for t0, n in ranges:
            def fresh(l):
                return tuple(U.bits_to_torch(x[t0:t0 + n]) for x in host[l])     # new device tensors, dropped after the call
            driver.block(t0, fresh)
            # churn the caching allocator: tensors of the sizes just dropped, overwritten at once
            junk = [torch.full((n, wl.n_kv_heads, wl.head_dim), float("nan"), dtype=torch.bfloat16, device=DEV)
                    for _ in range(2 * layers)]
            del junk
        driver.finish()
        torch.cuda.synchronize()
        st = []
        for l in range(layers):
            k, v, idx, w, count, nxt = cache.decode_ready(l)
            st.append((k[:, :count].clone(), v[:, :count].clone(), idx[:, :count].clone(), w[:, :count].clone()))
        results.append(st)
        cache.close()
    for a, b in zip(*results):
        for x, y in zip(a, b):
            assert torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x,
                               y.view(torch.int16) if y.dtype == torch.bfloat16 else y)

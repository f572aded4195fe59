"""GPU parity of the key-split bf16 attention kernel (small launches) at the edges of its
tiling: 16- and 32-query workgroups, 32-key blocks dealt over eight waves, read sets with
fewer blocks than waves, segments that end inside a block; single, batched and packed
launches (the packed one with its log-sum-exp).  Bars of the bf16 path: max-abs 2e-2 and
relative-L2 5e-3 of float64 per call; log-sum-exp within 1e-4 (float32 sums of at most 300
probabilities, each with a relative error of a few 2^-24 times the score's magnitude)."""
import math

import numpy as np
import pytest
import torch

import synth
from oracle import ff_oracle as fo
from paper_2609_32540_amd import ff

from gpu_util import PairedRun, check_attention, exact, last_launch, make_cache, make_oracle, to_dev
from test_gpu_packed import clip, oracle_packed
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ff.lib()


# chunk tokens 3, 15, 18, 33 and 99 (16-query workgroups), and 351 with 24 heads (528
# workgroups of one tile are three rounds: two tiles a workgroup, the last ragged, from 16 key
# tiles on, at d = 64 from 22; its first call, of 10, is left to the 256-query kernel)
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,grid", [(1, (1, 1)), (2, (1, 5)), (2, (2, 3)), (3, (1, 11)), (3, (3, 11)),
                                        (24, (9, 13))])
def test_tiles_and_blocks(head_dim, heads, grid):
    w = small("bf16", head_dim, heads=heads, grid_h=grid[0], grid_w=grid[1], stages=1, layers=1,
              n_chunks=4)
    run = PairedRun(w, rope=False)
    for c in range(w.n_chunks):
        run.step(c, 0, 0)
        assert last_launch().query_tiles == (1 if heads < 24 else [0, 2 if head_dim == 128 else 1, 2, 2][c])


@pytest.mark.parametrize("head_dim", [64, 128])
def test_rising_scores(head_dim):
    # keys of later chunks scaled by 3^c: the reference max is raised again and again
    w = small("bf16", head_dim, grid_h=3, grid_w=7, stages=1, layers=1, n_chunks=4)
    cache, oracle = make_cache(w, 1, 1), make_oracle(w, 1, 1)
    for c in range(w.n_chunks):
        q, k, v = (synth.chunk_tensor(w, t, c, 0, 0) for t in (synth.T_Q, synth.T_K, synth.T_V))
        k = (k.float() * 3.0 ** c).to(k.dtype)
        out = cache.chunk_attention(0, 0, c, to_dev(q), to_dev(k), to_dev(v))
        check_attention(exact(out), oracle.attention(0, 0, c, exact(q), exact(k), exact(v)), "bf16",
                        f"chunk {c}")
        cache.kv_publish(0, 0, c, to_dev(k), to_dev(v))
        oracle.publish(0, 0, c, exact(k), exact(v))


@pytest.mark.parametrize("head_dim", [64, 128])
def test_batch_items_of_different_lengths(head_dim):
    w = small("bf16", head_dim, grid_h=5, grid_w=7, ring_chunks=3, stages=3, layers=1, n_chunks=3)
    cache, oracle = make_cache(w, 3, 1), make_oracle(w, 3, 1)
    items = []
    for s in range(3):     # stage s holds s chunks
        for c in range(s + 1):
            q, k, v = (to_dev(synth.chunk_tensor(w, t, c, s, 0)) for t in (synth.T_Q, synth.T_K, synth.T_V))
            if c < s:
                cache.kv_publish(s, 0, c, k, v)
                oracle.publish(s, 0, c, exact(k), exact(v))
        items.append(dict(stage=s, layer=0, chunk=s, q=q, k=k, v=v))
    outs = cache.chunk_attention_batch(items)
    assert last_launch().query_tiles == 1
    for s, (it, out) in enumerate(zip(items, outs)):
        ref = oracle.attention(s, 0, s, exact(it["q"]), exact(it["k"]), exact(it["v"]))
        check_attention(exact(out), ref, "bf16", f"stage {s}")


# An item has the bits of its single call without a workspace whatever the other items are,
# also where the two launches would do best with different forms: 16 queries a workgroup alone
# and 32 in a batch of four (6 heads x 351 queries over 1053 keys, 12 x 198 over 1024, 24 x 198
# at d = 64); the key-split kernel alone and the 256-query one in a batch (24 x 351, 40 x 198,
# 12 x 1170); items on both sides of the line in one batch (38 x 198 at d = 64: 4 key tiles
# against 8 and 12).  With scratch too where there are fewer than 16 key tiles.
@pytest.mark.parametrize("heads,grid,head_dim,W", [(6, (9, 13), 128, 2), (12, (6, 11), 128, 3),
                                                   (24, (6, 11), 64, 2), (24, (9, 13), 128, 2),
                                                   (40, (6, 11), 128, 1), (12, (15, 26), 128, 3),
                                                   (12, (15, 26), 64, 3), (38, (6, 11), 64, 2)])
def test_batch_items_have_the_bits_of_their_single_calls(heads, grid, head_dim, W):
    S = 4
    w = small("bf16", head_dim, heads=heads, grid_h=grid[0], grid_w=grid[1], ring_chunks=W, stages=S,
              layers=1, n_chunks=W + 1)
    cache, g = make_cache(w, S, 1), torch.Generator(device="cuda").manual_seed(heads)
    rnd = lambda: torch.randn((w.chunk_tokens, heads, head_dim), generator=g, device="cuda").to(torch.bfloat16)
    items = []
    for s in range(S):      # stage 0 holds no chunk, stage 3 a full ring
        n = s * W // (S - 1)
        for c in range(n):
            cache.kv_publish(s, 0, c, rnd(), rnd())
        items.append(dict(stage=s, layer=0, chunk=n, q=rnd(), k=rnd(), v=rnd()))
    singles = [cache.chunk_attention_ws(it["stage"], 0, it["chunk"], it["q"], it["k"], it["v"], None)
               for it in items]
    for it, one in zip(items, singles):
        if (it["chunk"] + 1) * -(-w.chunk_tokens // 64) < 16:
            assert torch.equal(one, cache.chunk_attention(it["stage"], 0, it["chunk"], it["q"], it["k"], it["v"]))
    for pick in ([0, 1, 2, 3], [0, 3], [2], [1, 1, 1]):
        outs = cache.chunk_attention_batch([dict(items[j], out=torch.empty_like(items[j]["q"])) for j in pick])
        for j, out in zip(pick, outs):
            assert torch.equal(out, singles[j]), (pick, j)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("grid", [(1, 1), (3, 5), (5, 7)])
def test_packed_with_log_sum_exp(head_dim, grid):
    w = small("bf16", head_dim, grid_h=grid[0], grid_w=grid[1], stages=1, layers=1, n_chunks=4)
    n, G = 4, w.tokens_per_frame
    q, k, v = (to_dev(t) for t in clip(w, n))
    ak, av = (to_dev(t) for t in synth.anchor_tensors(w, [0, 1, 2], 0))
    table = [[0], [2, 0], [], [0, 1, 2]]
    lse = torch.empty(q.shape[:2], dtype=torch.float32, device=q.device)
    scale = 1.0 / math.sqrt(head_dim)
    out = ff.packed_attention(q, k, v, n_chunks=n, window=1, anchor_k=ak, anchor_v=av, frame_tokens=G,
                              anchors_of_chunk=table, lse=lse)
    assert last_launch().query_tiles == 1
    ref = oracle_packed(w, q, k, v, ak, av, table, 1, scale)
    nq = w.chunk_tokens
    for c in range(n):
        check_attention(exact(out[c * nq:(c + 1) * nq]), ref[c], "bf16", f"chunk {c}")
        keys = [exact(ak[f * G:(f + 1) * G]) for f in table[c]] + [exact(k[max(0, c - 1) * nq:(c + 1) * nq])]
        keys = np.concatenate(keys)
        want = fo.log2_sum_exp2(exact(q[c * nq:(c + 1) * nq]), keys, np.ones((nq, len(keys)), bool), scale)
        np.testing.assert_allclose(exact(lse[c * nq:(c + 1) * nq]), want, atol=1e-4)


def rounded_like_the_256_query_kernel(q, K, V, scale):
    """Attention with the probabilities rounded to bf16 relative to the reference that the
    256-query kernel starts from, the largest score of the first 32 keys, and normalised by
    their sum (float64 otherwise; the output rounded to bf16)."""
    out = torch.empty(q.shape, dtype=torch.float64)
    for h in range(q.shape[1]):
        s = (q[:, h].double() @ K[:, h].double().T) * (scale / math.log(2.0))
        p = torch.exp2(s - s[:, :32].max(1, keepdim=True).values).to(torch.bfloat16).double()
        out[:, h] = (p @ V[:, h].double()) / p.sum(1, keepdim=True)
    return out.to(torch.bfloat16).float().numpy()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_probabilities_are_rounded_as_by_the_256_query_kernel(head_dim):
    # A float32 score is off by a few 2^-24 of its size (up to 10 here), which moves about one
    # probability in 2000 across a rounding border, by 2^-8 of it: relative-L2 about 1e-4.
    # Rounded relative to another reference, every probability differs by up to 2^-8: 3e-3.
    w = small("bf16", head_dim, grid_h=6, grid_w=11, stages=1, layers=1, n_chunks=2)
    cache, K, V = make_cache(w, 1, 1), [], []
    for c in range(w.n_chunks):
        q, k, v = (synth.chunk_tensor(w, t, c, 0, 0) for t in (synth.T_Q, synth.T_K, synth.T_V))
        out = exact(cache.chunk_attention(0, 0, c, to_dev(q), to_dev(k), to_dev(v)))
        K, V = K + [k], V + [v]
        ref = rounded_like_the_256_query_kernel(q, torch.cat(K), torch.cat(V), 1.0 / math.sqrt(head_dim))
        assert np.linalg.norm(out - ref) <= 5e-4 * np.linalg.norm(ref)
        cache.kv_publish(0, 0, c, to_dev(k), to_dev(v))


@pytest.mark.parametrize("head_dim", [64, 128])
def test_blocks_of_keys_that_score_minus_infinity(head_dim):
    # products past the float32 range: whole 32-key blocks, the first one of several waves
    # among them (and, in the second call, the read set's first), score -inf for every query
    # and get weight 0
    w = small("bf16", head_dim, grid_h=6, grid_w=11, stages=1, layers=1, n_chunks=1)
    q, k, v = (synth.chunk_tensor(w, t, 0, 0, 0) for t in (synth.T_Q, synth.T_K, synth.T_V))
    q[:, :, 0] = 1e25
    k[:, :, 0] = 0.0
    for dead in (np.r_[32:64, 96:160], np.r_[0:64, 192:198]):
        kk = k.clone()
        kk[dead, :, 0] = -1e25
        cache, oracle = make_cache(w, 1, 1), make_oracle(w, 1, 1)
        out = cache.chunk_attention(0, 0, 0, to_dev(q), to_dev(kk), to_dev(v))
        check_attention(exact(out), oracle.attention(0, 0, 0, exact(q), exact(kk), exact(v)), "bf16")


# launches left to the 256-query kernel, whose partial last round runs as 2, 3 and 4 key parts:
# 96, 80 and 60 units on 256 CUs
@pytest.mark.parametrize("heads,grid,head_dim,parts", [(24, (12, 22), 128, 2), (24, (12, 22), 64, 2),
                                                       (16, (15, 26), 128, 3), (12, (15, 26), 128, 4),
                                                       (12, (15, 26), 64, 4)])
def test_key_parts_of_the_256_query_kernel(heads, grid, head_dim, parts):
    w = small("bf16", head_dim, heads=heads, grid_h=grid[0], grid_w=grid[1], ring_chunks=5, stages=1,
              layers=1, n_chunks=6)
    run = PairedRun(w, rope=False)
    rows = np.r_[0:40, w.chunk_tokens - 40:w.chunk_tokens]
    for c in range(w.n_chunks):
        run.step(c, 0, 0, check=c >= 4, heads=[0, heads - 1], rows=rows)
        if c >= 4:
            assert last_launch()[:2] == (0, parts)

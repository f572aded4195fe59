"""GPU parity of the float32 attention kernel at the edges of its tiling: 16-query
tiles (one or two per workgroup, by the launch size), 16-key blocks dealt over eight
waves, read sets with fewer blocks than waves, segments that end inside a block, and
the single, batched and packed launches.  Bar: max-abs and relative-L2 1e-5 of float64."""
import numpy as np
import pytest
import torch

import synth
from paper_2609_32540_amd import ff

from gpu_util import PairedRun, check_attention, exact, make_cache, make_oracle, to_dev
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ff.lib()


# (heads, grid): chunk tokens 3 (one query tile, one block a segment), 15 and 18 (a tile
# less one row, a tile and two), 33, and 189 (12 tiles of 24 heads = 288 workgroups of one
# tile: the launch takes two tiles a workgroup, the last of them ragged)
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,grid", [(1, (1, 1)), (2, (1, 5)), (2, (2, 3)), (3, (1, 11)), (24, (7, 9))])
def test_tiles_and_blocks(head_dim, heads, grid):
    w = small("f32", head_dim, heads=heads, grid_h=grid[0], grid_w=grid[1], stages=1, layers=1,
              n_chunks=4)
    run = PairedRun(w, rope=False)
    for c in range(w.n_chunks):
        run.step(c, 0, 0)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_batch_equals_single_calls(head_dim):
    # bit-identical: a query's sums do not depend on the query tiles of its workgroup
    w = small("f32", head_dim, grid_h=5, grid_w=7, stages=3, layers=1, n_chunks=3)
    cache, oracle = make_cache(w, 3, 1), make_oracle(w, 3, 1)
    for c in range(w.n_chunks):
        items = []
        for s in range(3):
            q, k, v = (to_dev(synth.chunk_tensor(w, t, c, s, 0)) for t in (synth.T_Q, synth.T_K, synth.T_V))
            items.append(dict(stage=s, layer=0, chunk=c, q=q, k=k, v=v))
        outs = cache.chunk_attention_batch(items)
        for s, it in enumerate(items):
            one = cache.chunk_attention(s, 0, c, it["q"], it["k"], it["v"])
            assert torch.equal(one, outs[s])
            check_attention(exact(one), oracle.attention(s, 0, c, exact(it["q"]), exact(it["k"]),
                                                         exact(it["v"])), "f32", f"chunk {c} stage {s}")
            cache.kv_publish(s, 0, c, it["k"], it["v"])
            oracle.publish(s, 0, c, exact(it["k"]), exact(it["v"]))


@pytest.mark.parametrize("scale", [1e-3, 4.0])
def test_flat_and_peaked_rows(scale):
    # 4.0 times the raw products (|s| up to about 150): the running max moves many times and
    # most probabilities underflow.  Bar: a float32 score of magnitude S carries an error of
    # about 3 S 2^-24, the relative error of its probability (S = 150: 3e-5), so max-abs and
    # relative-L2 are bounded by 1e-4 there.
    w = small("f32", 64, stages=1, layers=1, n_chunks=3)
    cache, oracle = make_cache(w, 1, 1), make_oracle(w, 1, 1)
    for c in range(w.n_chunks):
        q, k, v = (synth.chunk_tensor(w, t, c, 0, 0) for t in (synth.T_Q, synth.T_K, synth.T_V))
        out = exact(cache.chunk_attention(0, 0, c, to_dev(q), to_dev(k), to_dev(v), scale=scale))
        ref = oracle.attention(0, 0, c, exact(q), exact(k), exact(v), scale=scale)
        bar = 1e-4 if scale > 1 else 1e-5
        err = np.abs(out - ref)
        assert err.max() <= bar and np.linalg.norm(err) <= bar * np.linalg.norm(ref)
        cache.kv_publish(0, 0, c, to_dev(k), to_dev(v))
        oracle.publish(0, 0, c, exact(k), exact(v))


@pytest.mark.parametrize("head_dim", [64, 128])
def test_infinite_value_in_a_segments_last_row(head_dim):
    # 27-token chunks end inside a 16-key block: its missing keys must add nothing, also where
    # the last row of V, which their addresses repeat, is infinite
    w = small("f32", head_dim, grid_h=3, grid_w=3, stages=1, layers=1, n_chunks=2)
    cache = make_cache(w, 1, 1)
    q, k, v = (to_dev(synth.chunk_tensor(w, t, 0, 0, 0)) for t in (synth.T_Q, synth.T_K, synth.T_V))
    v[-1, :, 3] = float("inf")
    out = cache.chunk_attention(0, 0, 0, q, k, v)
    assert torch.isinf(out[:, :, 3]).all()
    keep = [e for e in range(head_dim) if e != 3]
    oracle = make_oracle(w, 1, 1)
    vv = exact(v)
    vv[-1, :, 3] = 0.0
    ref = oracle.attention(0, 0, 0, exact(q), exact(k), vv)
    check_attention(exact(out)[..., keep], ref[..., keep], "f32")


def test_scores_are_scaled_before_they_are_summed():
    # |q.k| would pass the float32 range, scale * |q.k| does not
    w = small("f32", 64, grid_h=3, grid_w=3, stages=1, layers=1, n_chunks=2)
    cache, oracle = make_cache(w, 1, 1), make_oracle(w, 1, 1)
    q, k, v = (synth.chunk_tensor(w, t, 0, 0, 0) for t in (synth.T_Q, synth.T_K, synth.T_V))
    out = cache.chunk_attention(0, 0, 0, to_dev(q * 1e20), to_dev(k * 1e20), to_dev(v), scale=2.0 ** -135)
    ref = oracle.attention(0, 0, 0, exact(q * 1e20), exact(k * 1e20), exact(v), scale=2.0 ** -135)
    check_attention(exact(out), ref, "f32")


@pytest.mark.parametrize("head_dim", [64, 128])
def test_very_large_scores(head_dim):
    # scores of about 1e10 times N(0, 1): each row is one-hot on its largest key (float32 sums
    # of 64 to 128 products are off by under 1e5 there, the two largest of 27 to 81 scores are
    # 1e6 or more apart), so the output is that key's row of V to float32 rounding
    w = small("f32", head_dim, grid_h=3, grid_w=3, stages=1, layers=1, n_chunks=3)
    cache, hist = make_cache(w, 1, 1), []
    for c in range(w.n_chunks):
        q, k, v = (synth.chunk_tensor(w, t, c, 0, 0) for t in (synth.T_Q, synth.T_K, synth.T_V))
        q = q * 1e10
        out = exact(cache.chunk_attention(0, 0, c, to_dev(q), to_dev(k), to_dev(v)))
        hist.append((k.double(), v))
        K, V = (torch.cat([h[i] for h in hist]) for i in (0, 1))
        s = torch.einsum("qhd,khd->hqk", q.double(), K) / head_dim ** 0.5
        top = s.topk(2, dim=2)
        assert float((top.values[..., 0] - top.values[..., 1]).min()) > 1e6
        ref = torch.stack([V[top.indices[h, :, 0], h] for h in range(w.heads)], 1)
        np.testing.assert_allclose(out, ref.numpy(), rtol=1e-6, atol=0)
        cache.kv_publish(0, 0, c, to_dev(k), to_dev(v))


@pytest.mark.parametrize("head_dim", [64, 128])
def test_blocks_of_keys_that_score_minus_infinity(head_dim):
    # products past the float32 range: whole 16-key blocks, the read set's first one and the
    # first of several waves among them, score -inf for every query and get weight 0
    w = small("f32", head_dim, grid_h=6, grid_w=11, stages=1, layers=1, n_chunks=1)
    cache, oracle = make_cache(w, 1, 1), make_oracle(w, 1, 1)
    q, k, v = (synth.chunk_tensor(w, t, 0, 0, 0) for t in (synth.T_Q, synth.T_K, synth.T_V))
    q[:, :, 0] = 1e25
    k[:, :, 0] = 0.0
    dead = np.r_[0:16, 48:80, 128:144]
    k[dead, :, 0] = -1e25
    out = cache.chunk_attention(0, 0, 0, to_dev(q), to_dev(k), to_dev(v))
    check_attention(exact(out), oracle.attention(0, 0, 0, exact(q), exact(k), exact(v)), "f32")

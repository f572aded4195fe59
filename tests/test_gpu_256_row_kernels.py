"""GPU parity of the 256-query attention kernel and the 256-row backward kernels at sizes that
the launch choices leave to them, in the situations the smaller tests are about but reach with
the key-split kernels: the checked pass after an overflow of the fast one (single, batched and
packed launches, key parts, the waves without queries of a ragged last tile), key parts in a
caller's workspace, three key parts, concurrent tail splits, and the backward of peaked rows,
hidden frames and frames seen by several runs of chunks.  Every test asserts the form that the
launch took.  Mostly 12 heads x 1170 queries: 60 units of 256 queries, the last of a head with
146, so three of its eight waves have none.  Sampled rows and heads; bars of the bf16 path."""
import math

import numpy as np
import pytest
import torch

import synth
from oracle import ff_oracle as fo
from paper_2609_32540_amd import ff

from gpu_util import check_attention, exact, last_launch, make_cache, to_dev
from test_gpu_backward import TABLE6, run_case
from test_gpu_parity import small
from test_gpu_wavefront import make_stub

pytestmark = pytest.mark.gpu

HEADS, GRID = 12, (15, 26)
ROWS = np.r_[0:24, 500:524, 1000:1024, 1120:1170]   # the last tile holds queries 1024 .. 1169


@pytest.fixture(autouse=True, scope="module")
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ff.lib()


def workload(head_dim, W, heads=HEADS, **kw):
    base = dict(heads=heads, grid_h=GRID[0], grid_w=GRID[1], ring_chunks=W, stages=1, layers=1,
                n_chunks=W + 1, anchor_rule="none", max_anchor_frames=1)
    base.update(kw)
    return small("bf16", head_dim, **base)


def tensors(w, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn((w.chunk_tokens, w.heads, w.head_dim), generator=g, device="cuda").to(torch.bfloat16)
            for _ in range(3)]


# key scale of chunk c, a number or one per token: the fast pass keeps the column max of the
# first block it reads as its reference, and row sums past 2^64 of it send the unit through the
# checked pass
KEY_SCALES = {
    "rising": lambda w, c: [1.0, 3.0, 9.0, 27.0, 1.0 / 64][c],      # the max moves again and again
    "far": lambda w, c: [0.01, 8.0, 8.0, 24.0, 1.0][c],             # 2^35 and past 2^64 above the reference
    "halves": lambda w, c: torch.where(torch.arange(w.chunk_tokens, device="cuda") < w.chunk_tokens // 2,
                                       0.01, 24.0)[:, None, None],  # past it in every key part
}


def scaled(k, f):
    return (k.float() * f).to(torch.bfloat16)


def check_rows(out, q, keys, vals, what, rows=ROWS, heads=None):
    K, V = torch.cat(keys), torch.cat(vals)
    scale = 1.0 / math.sqrt(q.shape[2])
    for h in heads or (0, q.shape[1] - 1):
        ref = fo.attend(exact(q[rows, h]).astype(np.float64), exact(K[:, h]).astype(np.float64),
                        exact(V[:, h]).astype(np.float64), scale)
        check_attention(exact(out[rows, h]), ref, "bf16", f"{what} head {h}")


def row_sums(q, keys):
    """Row sums relative to the first 32 keys' largest score, log2, of the sampled rows of head 0."""
    K = torch.cat(keys)[:, 0].double()
    s = q[ROWS, 0].double() @ K.T * (math.log2(math.e) / math.sqrt(q.shape[2]))
    return torch.logsumexp((s - s[:, :32].max(1, keepdim=True).values) * math.log(2.0), 1) / math.log(2.0)


@pytest.mark.parametrize("head_dim", [128, 64])
@pytest.mark.parametrize("scratch", [True, False])
@pytest.mark.parametrize("keys", sorted(KEY_SCALES))
def test_checked_pass_of_a_single_launch(head_dim, scratch, keys):
    w = workload(head_dim, 4)
    cache, hist, overflows = make_cache(w, 1, 1), [], 0
    for c in range(w.n_chunks):
        q, k, v = tensors(w, 100 + c)
        k = scaled(k, KEY_SCALES[keys](w, c))
        if scratch:
            out = cache.chunk_attention(0, 0, c, q, k, v)
        else:
            out = cache.chunk_attention_ws(0, 0, c, q, k, v, None)
        form = last_launch()[:2]
        cache.kv_publish(0, 0, c, k, v)
        hist.append((k, v))
        K, V = [h[0] for h in hist], [h[1] for h in hist]
        check_rows(out, q, K, V, f"chunk {c}")
        if not scratch:
            assert form == (0, 1)
            overflows += int((row_sums(q, K) > 70).any())
        elif c >= 2:
            assert form == (0, 4)
    assert scratch or overflows >= (1 if keys == "rising" else 2)


@pytest.mark.parametrize("head_dim", [128, 64])
def test_checked_pass_of_a_batch(head_dim):
    S, W = 4, 2
    w = workload(head_dim, W, stages=S)
    cache, items, read = make_cache(w, S, 1), [], []
    for s in range(S):
        K, V = [], []
        for c in range(min(s, W) + 1):
            q, k, v = tensors(w, 10 * s + c)
            k = scaled(k, KEY_SCALES["halves"](w, c) if s != 1 else 1.0)   # item 1: no overflow
            K.append(k), V.append(v)
            if c < min(s, W):
                cache.kv_publish(s, 0, c, k, v)
        assert bool((row_sums(q, K) > 70).any()) == (s != 1)
        items.append(dict(stage=s, layer=0, chunk=len(K) - 1, q=q, k=k, v=v))
        read.append((K, V))
    outs = cache.chunk_attention_batch(items)
    assert last_launch().query_tiles == 0
    for s, (it, out, (K, V)) in enumerate(zip(items, outs, read)):
        check_rows(out, it["q"], K, V, f"stage {s}")


@pytest.mark.parametrize("head_dim", [128, 64])
@pytest.mark.parametrize("with_lse", [True, False])
def test_checked_pass_of_a_packed_launch(head_dim, with_lse):
    n, W = 5, 4
    w = workload(head_dim, W)
    parts = [tensors(w, 200 + c) for c in range(n)]
    for c, p in enumerate(parts):
        p[1] = scaled(p[1], KEY_SCALES["far"](w, c))
    q, k, v = (torch.cat([p[i] for p in parts]) for i in range(3))
    lse = torch.empty(q.shape[:2], dtype=torch.float32, device="cuda") if with_lse else None
    out = ff.packed_attention(q, k, v, n_chunks=n, window=W, lse=lse)
    assert last_launch().query_tiles == 0
    nq, scale = w.chunk_tokens, 1.0 / math.sqrt(head_dim)
    for c in range(n):
        K, V = [p[1] for p in parts[:c + 1]], [p[2] for p in parts[:c + 1]]
        check_rows(out[c * nq:(c + 1) * nq], parts[c][0], K, V, f"chunk {c}")
        if with_lse:
            Kh = torch.cat(K)[:, :1]
            want = fo.log2_sum_exp2(exact(parts[c][0][ROWS][:, :1]), exact(Kh),
                                    np.ones((len(ROWS), Kh.shape[0]), bool), scale)
            # (2e-3 log2 units: bar of the backward's log-sum-exp)
            assert np.abs(exact(lse[c * nq + ROWS, :1]) - want).max() <= 2e-3
    assert bool((row_sums(parts[3][0], [p[1] for p in parts[:4]]) > 70).any())


def test_three_key_parts():
    # 16 heads x 5 tiles = 80 units: three parts fill 240 of the 256 compute units
    w = workload(128, 4, heads=16)
    cache, hist = make_cache(w, 1, 1), []
    for c in range(w.n_chunks):
        q, k, v = tensors(w, 300 + c)
        out = cache.chunk_attention(0, 0, c, q, k, v)
        if c >= 2:
            assert last_launch()[:2] == (0, 3)
        cache.kv_publish(0, 0, c, k, v)
        hist.append((k, v))
        check_rows(out, q, [h[0] for h in hist], [h[1] for h in hist], f"chunk {c}")


@pytest.mark.parametrize("head_dim", [128, 64])
def test_two_layers_of_one_stage_with_key_parts_in_two_workspaces(head_dim):
    # both layers' key parts in flight at once; the partial results go to the callers'
    # workspaces (poisoned before) and none to the cache's own scratch (the end of its buffer)
    w = workload(head_dim, 3, layers=2)
    cache, plain = make_cache(w, 1, 2), make_cache(w, 1, 2)
    n_ws = cache.workspace_bytes()
    own = cache.buffer[cache.buffer.numel() - n_ws:]
    own.fill_(0xFF)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    workspaces = [torch.empty(n_ws, dtype=torch.uint8, device="cuda") for _ in streams]
    hist = [[], []]
    for c in range(w.n_chunks):
        inputs = [tensors(w, 400 + 10 * c + l) for l in (0, 1)]
        for ws in workspaces:
            ws.fill_(0xFF)
        torch.cuda.synchronize()
        outs, forms = [], []
        for l, (q, k, v) in enumerate(inputs):
            outs.append(cache.chunk_attention_ws(0, l, c, q, k, v, workspaces[l], stream=streams[l]))
            forms.append(last_launch()[:2])
            cache.kv_publish(0, l, c, k, v, stream=streams[l])
        torch.cuda.synchronize()
        for l, (q, k, v) in enumerate(inputs):
            hist[l].append((k, v))
            check_rows(outs[l], q, [h[0] for h in hist[l]], [h[1] for h in hist[l]], f"chunk {c} layer {l}")
            if c >= 2:
                assert forms[l] == (0, 4)
                assert bool((workspaces[l] != 0xFF).any())
            assert torch.equal(plain.chunk_attention(0, l, c, q, k, v), outs[l])
            plain.kv_publish(0, l, c, k, v)
    assert bool((own == 0xFF).all())


def test_workspace_sizes_limit_the_key_parts():
    # 4 parts of 60 units; where half the workspace leaves two, the key-split kernel is faster
    w = workload(128, 3)
    n_ws = make_cache(w, 1, 1).workspace_bytes()
    sizes = [(n_ws, (0, 4)), (n_ws // 2, (2, 1)), (n_ws // 3, (0, 1)), (0, (0, 1))]
    caches = [make_cache(w, 1, 1) for _ in sizes]
    hist = []
    for c in range(w.n_chunks):
        q, k, v = tensors(w, 500 + c)
        hist.append((k, v))
        for cache, (n, form) in zip(caches, sizes):
            ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
            out = cache.chunk_attention_ws(0, 0, c, q, k, v, ws)
            if c >= 2:
                assert last_launch()[:2] == form
            cache.kv_publish(0, 0, c, k, v)
            check_rows(out, q, [h[0] for h in hist], [h[1] for h in hist], f"chunk {c} workspace {n}")


@pytest.mark.parametrize("head_dim", [128, 64])
def test_batch_items_beside_single_calls_with_key_parts(head_dim):
    # a batch has no key parts: equal within the bar, not bitwise
    S, W = 2, 3
    w = workload(head_dim, W, stages=S)
    cache, read, items = make_cache(w, S, 1), [], []
    for s in range(S):
        chunks = [tensors(w, 600 + 10 * s + c) for c in range(W + 1)]
        for c in range(W):
            cache.kv_publish(s, 0, c, chunks[c][1], chunks[c][2])
        read.append(([t[1] for t in chunks], [t[2] for t in chunks]))
        items.append(dict(stage=s, layer=0, chunk=W, q=chunks[W][0], k=chunks[W][1], v=chunks[W][2]))
    outs = cache.chunk_attention_batch(items)
    assert last_launch()[:2] == (0, 1)
    for s, it in enumerate(items):
        one = cache.chunk_attention(s, 0, W, it["q"], it["k"], it["v"])
        assert last_launch()[:2] == (0, 4)
        check_rows(one, it["q"], *read[s], f"single stage {s}")
        check_rows(outs[s], it["q"], *read[s], f"batch stage {s}")


def test_wavefront_with_concurrent_key_parts():
    # four stages on four streams, each with its key parts in its own scratch: the latents
    # and rings of a chunk-major run on one stream, bit for bit
    S, N_R, W = 4, 4, 3
    w = workload(128, W, stages=S, n_chunks=N_R)
    results = []
    for wavefront in (False, True):
        cache = make_cache(w, S, 1)
        X = [tensors(w, 700 + i)[0] for i in range(N_R)]
        forward, forms = make_stub(cache, w, X, 1), set()

        def recorded(s, i, stream):
            forward(s, i, stream)
            forms.add(last_launch()[:2])
        torch.cuda.synchronize()
        if wavefront:
            ff.wavefront_run(N_R, [torch.cuda.Stream() for _ in range(S)], recorded)
        else:
            stream = torch.cuda.Stream()
            for i in range(N_R):
                for s in range(S):
                    recorded(s, i, stream)
        torch.cuda.synchronize()
        assert (0, 4) in forms
        results.append((X, [cache.read(s, 0, slot) for s in range(S) for slot in range(W)]))
    torch.cuda.synchronize()
    for a, b in zip(results[0][0], results[1][0]):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
    for (ka, va), (kb, vb) in zip(results[0][1], results[1][1]):
        assert torch.equal(ka, kb) and torch.equal(va, vb)


# 250-token chunks: one ragged 256-row tile each; heads enough for 256-row kernels in both passes
@pytest.mark.parametrize("d,heads", [(128, 24), (64, 40)])
@pytest.mark.parametrize("case", ["peaked", "hidden frame"])
def test_backward(d, heads, case):
    if case == "peaked":     # keys scaled by 6: P close to one-hot for many rows
        run_case(6, 250, 70, 3, TABLE6, 2, heads, d, seed=41, key_scale=6.0)
    else:
        run_case(6, 250, 70, 4, [[0], [0, 1], [1], [1, 3], [3], [3]], 3, heads, d, seed=43, hidden_frame=True)
    assert last_launch()[2:] == (0, 0)


@pytest.mark.parametrize("d,heads,Nq,G", [(128, 24, 250, 70), (64, 32, 500, 64)])
def test_backward_frame_seen_by_several_chunk_runs(d, heads, Nq, G):
    # frame 0 is seen by chunks {0, 1, 3, 5}: three runs of consecutive chunks
    run_case(6, Nq, G, 2, [[0], [0], [1], [0, 1], [1], [0]], 1, heads, d, seed=45)
    assert last_launch()[2:] == (0, 0)
